// dms_gradient.hip -- discrete gradient by Robins et al.'s ProcessLowerStars,
// one GPU thread per vertex (Section 2.3: the gradient is computed by
// inspecting the local neighbourhood of each vertex, which makes the step
// embarrassingly parallel; cells are compared as in Section 2.1).
//
// Most vertices of a smooth field take their record from tables indexed by
// their lower neighbours and the order of those (see table_entry).  Any other
// vertex is solved from its sorted neighbours by two growing forests that
// give Robins' pairing without its queues (see solve_star).  k_gradient does
// the table vertices of every tile and hands the others over: a tile with few
// of them queues them (k_gradient_queue), a tile with many is listed whole
// (k_gradient_dense).
// The outcome is packed into the 16-byte record described in dms.h.
// Readings: "unpaired" = neither paired nor critical; only unpaired cells
// enter the one-facet queue; entries of the zero queue that get paired are
// dropped (Robins' lazy deletion gives the same pops).
#include <atomic>
#include <mutex>

#include "dms_common.hpp"
#include "dms_internal.hpp"
#include "dms_tables.hpp"

namespace dms {
namespace {

constexpr int kThreads = 256;      // threads per block
constexpr int kTileVerts = 1024;  // vertices per tile (4 per thread)
constexpr int32_t kAbsent = 0x7fffffff;

// Tables of solve_star, staged in LDS (9 KB).  Everything is relative to a
// vertex's lowest neighbour d: once x is paired with the edge to d, every
// lower triangle through d is paired too, so only the star triangles that do
// not contain d are searched -- at most 32 of the 36 (each neighbour lies on
// 4 or 6), one 32-bit word.  "Triangle bit" below is a triangle's position
// among those, in star order.
struct StarTables {
    // [d][e]: triangle bits containing neighbour e; [d][14]: the unused bits;
    // [d][15]: star tets containing d
    alignas(16) uint32_t tris[14][16];
    // [d][bit]: low word = the star tets containing the triangle, star index
    // of the triangle << 24; high word = a | field(a) << 4 | b << 8 |
    // field(b) << 12 for its neighbours a, b, field(e) = the record field of
    // edge e when it is paired with this triangle
    alignas(16) uint64_t tri[14][32];
    // [d][q]: low word = triangle bits of tet q, high word = those of them
    // whose first star tet is q
    alignas(16) uint64_t tet[14][24];
    // [2 t + v - 1]: the last three record words with triangle t's field = v
    alignas(16) uint32_t field[72][4];
    // [d]: edge fields with d paired with x and every neighbour of d in the
    // link paired with its triangle through d
    uint64_t fan[14];
    uint32_t nibbles[128];  // bit i -> 0xf << 4 i
    uint16_t link[16];
};

constexpr StarTables make_star_tables()
{
    StarTables S{};
    const Tables &T = kTables;
    for (int d = 0; d < 14; ++d) {
        int bit[36] = {}, n = 0;
        for (int t = 0; t < 36; ++t) bit[t] = T.tri[t][0] == d || T.tri[t][1] == d ? -1 : n++;
        S.tris[d][14] = n < 32 ? ~0u << n : 0u;
        S.tris[d][15] = T.edge_tetmask[d];
        for (int t = 0; t < 36; ++t) {
            const int a = T.tri[t][0], b = T.tri[t][1];
            const uint32_t fa = 3u + (uint32_t)T.tri_slot[t][0], fb = 3u + (uint32_t)T.tri_slot[t][1];
            if (bit[t] < 0) {
                const int o = a == d ? b : a;
                S.fan[d] |= (uint64_t)(o == a ? fa : fb) << (4 * o);
                continue;
            }
            S.tris[d][a] |= 1u << bit[t];
            S.tris[d][b] |= 1u << bit[t];
            const uint32_t ends = (uint32_t)a | fa << 4 | (uint32_t)b << 8 | fb << 12;
            S.tri[d][bit[t]] = (uint64_t)ends << 32 | (uint64_t)(T.tri_tetmask[t] | (uint32_t)t << 24);
        }
        S.fan[d] |= 1ull << (4 * d);
        for (int q = 0; q < 24; ++q)
            for (int c = 0; c < 3; ++c) {
                const int t = T.tet_tris[q][c];
                if (bit[t] < 0) continue;
                S.tet[d][q] |= 1ull << bit[t];
                if (T.tri_tets[t][0] == q) S.tet[d][q] |= 1ull << (32 + bit[t]);
            }
        S.link[d] = T.link[d];
    }
    for (int t = 0; t < 36; ++t)
        for (uint32_t v = 1; v <= 2; ++v) {
            const int at = 24 + 2 * t;  // from the record's second word
            S.field[2 * t + (int)v - 1][at / 32] = v << (at % 32);
        }
    for (uint32_t m = 0; m < 128; ++m)
        for (int i = 0; i < 7; ++i)
            if ((m >> i) & 1u) S.nibbles[m] |= 0xfu << (4 * i);
    return S;
}

__device__ const StarTables g_star = make_star_tables();
static_assert(sizeof(StarTables) % 16 == 0, "copied as 16-byte words");

__device__ __forceinline__ uint32_t nib(uint64_t packed, int i) { return (uint32_t)(packed >> (4 * i)) & 15u; }

// Comparison keys.  The gradient only compares x with its neighbours and
// the neighbours among themselves, in the order of Section 2.1: by value,
// ties by vertex id.  Ranks (the global order) are one encoding of it; the
// values themselves are another (the equivalent form that needs no sort).
//  RankKeys: the LDS halo holds int32 ranks, compared directly.
//  F32Keys / F64Keys: the halo holds order-preserving unsigned keys of the
//    values (-0.0 as +0.0); a comparison value is key << 4 | slot, where the
//    slot orders x and its neighbours by id (neighbours 0..6 precede x, 7..13
//    follow it), so equal values break ties by id.  The 36 bits of F32Keys
//    are held in a double, whose comparisons and minima are single
//    instructions at the rate of the 32-bit ones (64-bit integers have no
//    minimum instruction).
// Id-order slot of neighbour e relative to x (x itself is slot 7).
__device__ __forceinline__ constexpr int id_slot(int e) { return e < 7 ? e : e + 1; }

// The 36-bit integer high4 << 32 | low32 as a double (2^52 plus it, so that
// doubles compare like the integers).
__device__ __forceinline__ double packed36(uint32_t high4, uint32_t low32)
{
    return __longlong_as_double((long long)((uint64_t)(0x43300000u | high4) << 32 | low32));
}

// Minimum and maximum of two such doubles, in one instruction each (none is
// a NaN, which the language's own min and max would have to provide for).
__device__ __forceinline__ double min_packed(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double max_packed(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

template <typename C>
__device__ __forceinline__ C cmin(C a, C b) { return b < a ? b : a; }
template <>
__device__ __forceinline__ double cmin<double>(double a, double b) { return min_packed(a, b); }

// A comparison value above every real one.
template <typename C> __device__ __forceinline__ constexpr C c_highest();
template <> __device__ __forceinline__ constexpr int32_t c_highest<int32_t>() { return 0x7fffffff; }
template <> __device__ __forceinline__ constexpr double c_highest<double>() { return 9007199254740992.0; }
template <> __device__ __forceinline__ constexpr unsigned __int128 c_highest<unsigned __int128>()
{
    return ~(unsigned __int128)0;
}

struct RankKeys {
    using H = int32_t;
    using C = int32_t;
    static constexpr H kAbsentH = kAbsent;
    __device__ static H load(const void *f, int64_t i, bool &nan)
    {
        nan = false;
        return ((const int32_t *)f)[i];
    }
    __device__ static C cmp(H h, int) { return h; }
    // order << 4 | e, with the order's sign bit flipped (any int32 labelling)
    __device__ static double sort_key(C o, int e) { return packed36(((uint32_t)o >> 28) ^ 8u, (uint32_t)o << 4 | (uint32_t)e); }
    static constexpr bool kSlots = false;
};

struct F32Keys {
    using H = uint32_t;
    using C = double;
    static constexpr H kAbsentH = 0xffffffffu;  // a NaN's key: never a valid input, above every valid one
    __device__ static H load(const void *f, int64_t i, bool &nan) { return key_of(((const float *)f)[i], nan); }
    __device__ static C cmp(H h, int slot) { return packed36(h >> 28, h << 4 | (uint32_t)slot); }
    __device__ static double sort_key(C o, int) { return o; }
    static constexpr bool kSlots = true;  // the low four bits name the slot, not the neighbour
};

struct F64Keys {
    using H = uint64_t;
    using C = unsigned __int128;
    static constexpr H kAbsentH = ~0ull;
    __device__ static H load(const void *f, int64_t i, bool &nan) { return key_of(((const double *)f)[i], nan); }
    __device__ static C cmp(H h, int slot) { return h == kAbsentH ? c_highest<C>() : ((C)h << 4) | (C)slot; }
};

// Comparisons that are only counted or collected into a mask: the compare's
// lane mask goes to a scalar pair and from there into the carry of an addition,
// one vector instruction each (the compiler selects 0 or 1 by the mask, then
// ORs or adds, and fills the two wait states between a compare and the read of
// its mask with nops).  Three scalar pairs in turn put two other instructions
// between each compare and its use.  T: the comparison's type.
#define DMS_CMP(T, s, a, b) "v_cmp_lt_" T "_e64 %[s" #s "], %[" #a "], %[" #b "]\n\t"
#define DMS_BIT(l, s) "v_addc_co_u32_e64 %[" #l "], vcc, %[" #l "], %[" #l "], %[s" #s "]\n\t"  // l = 2 l + mask
#define DMS_INC(l, s) "v_addc_co_u32_e64 %[" #l "], vcc, 0, %[" #l "], %[s" #s "]\n\t"      // l = l + mask
#define DMS_SET(l, s) "v_cndmask_b32_e64 %[" #l "], 0, 1, %[s" #s "]\n\t"                   // l = mask

#define DMS_LOWER_MASK(T)                                                                                          \
    DMS_CMP(T, 0, o13, x) DMS_CMP(T, 1, o12, x) DMS_CMP(T, 2, o11, x) DMS_SET(l, 0)                                 \
    DMS_CMP(T, 0, o10, x) DMS_BIT(l, 1) DMS_CMP(T, 1, o9, x) DMS_BIT(l, 2)                                         \
    DMS_CMP(T, 2, o8, x) DMS_BIT(l, 0) DMS_CMP(T, 0, o7, x) DMS_BIT(l, 1)                                          \
    DMS_CMP(T, 1, o6, x) DMS_BIT(l, 2) DMS_CMP(T, 2, o5, x) DMS_BIT(l, 0)                                          \
    DMS_CMP(T, 0, o4, x) DMS_BIT(l, 1) DMS_CMP(T, 1, o3, x) DMS_BIT(l, 2)                                          \
    DMS_CMP(T, 2, o2, x) DMS_BIT(l, 0) DMS_CMP(T, 0, o1, x) DMS_BIT(l, 1)                                          \
    DMS_CMP(T, 1, o0, x) DMS_BIT(l, 2) "s_nop 0\n\t" DMS_BIT(l, 0) "s_nop 0\n\t" DMS_BIT(l, 1)

// Lower-neighbour mask of x: bit e set if neighbour e precedes x.
template <typename C>
__device__ __forceinline__ uint32_t lower_mask(const C *o, C ox)
{
    uint32_t low = 0;
    if constexpr (sizeof(C) > 8) {
#pragma unroll
        for (int e = 0; e < 14; ++e) low |= (o[e] < ox ? 1u : 0u) << e;
    } else {
        uint64_t s0, s1, s2;
#define DMS_OPERANDS                                                                                                \
    : [l] "=&v"(low), [s0] "=&s"(s0), [s1] "=&s"(s1), [s2] "=&s"(s2)                                                \
    : [x] "v"(ox), [o0] "v"(o[0]), [o1] "v"(o[1]), [o2] "v"(o[2]), [o3] "v"(o[3]), [o4] "v"(o[4]), [o5] "v"(o[5]),     \
      [o6] "v"(o[6]), [o7] "v"(o[7]), [o8] "v"(o[8]), [o9] "v"(o[9]), [o10] "v"(o[10]), [o11] "v"(o[11]),             \
      [o12] "v"(o[12]), [o13] "v"(o[13])                                                                            \
    : "vcc"
        if constexpr (sizeof(C) == 4) asm(DMS_LOWER_MASK("i32") DMS_OPERANDS);
        else asm(DMS_LOWER_MASK("f64") DMS_OPERANDS);
#undef DMS_OPERANDS
    }
    return low;
}

// Lehmer digits of eight values: l[i] = how many of the later ones are smaller.
#define DMS_DIGITS(T)                                                                                              \
    DMS_CMP(T, 0, v7, v6) DMS_CMP(T, 1, v7, v5) DMS_CMP(T, 2, v7, v4) DMS_SET(l6, 0)                                \
    DMS_CMP(T, 0, v7, v3) DMS_SET(l5, 1) DMS_CMP(T, 1, v7, v2) DMS_SET(l4, 2)                                      \
    DMS_CMP(T, 2, v7, v1) DMS_SET(l3, 0) DMS_CMP(T, 0, v7, v0) DMS_SET(l2, 1)                                      \
    DMS_CMP(T, 1, v6, v5) DMS_SET(l1, 2) DMS_CMP(T, 2, v6, v4) DMS_SET(l0, 0)                                      \
    DMS_CMP(T, 0, v6, v3) DMS_INC(l5, 1) DMS_CMP(T, 1, v6, v2) DMS_INC(l4, 2)                                      \
    DMS_CMP(T, 2, v6, v1) DMS_INC(l3, 0) DMS_CMP(T, 0, v6, v0) DMS_INC(l2, 1)                                      \
    DMS_CMP(T, 1, v5, v4) DMS_INC(l1, 2) DMS_CMP(T, 2, v5, v3) DMS_INC(l0, 0)                                      \
    DMS_CMP(T, 0, v5, v2) DMS_INC(l4, 1) DMS_CMP(T, 1, v5, v1) DMS_INC(l3, 2)                                      \
    DMS_CMP(T, 2, v5, v0) DMS_INC(l2, 0) DMS_CMP(T, 0, v4, v3) DMS_INC(l1, 1)                                      \
    DMS_CMP(T, 1, v4, v2) DMS_INC(l0, 2) DMS_CMP(T, 2, v4, v1) DMS_INC(l3, 0)                                      \
    DMS_CMP(T, 0, v4, v0) DMS_INC(l2, 1) DMS_CMP(T, 1, v3, v2) DMS_INC(l1, 2)                                      \
    DMS_CMP(T, 2, v3, v1) DMS_INC(l0, 0) DMS_CMP(T, 0, v3, v0) DMS_INC(l2, 1)                                      \
    DMS_CMP(T, 1, v2, v1) DMS_INC(l1, 2) DMS_CMP(T, 2, v2, v0) DMS_INC(l0, 0)                                      \
    DMS_CMP(T, 0, v1, v0) DMS_INC(l1, 1) "s_nop 0\n\t" DMS_INC(l0, 2) "s_nop 0\n\t" DMS_INC(l0, 0)

template <typename C>
__device__ __forceinline__ void lehmer_digits(const C *v, uint32_t *l)
{
    if constexpr (sizeof(C) > 8) {
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            l[i] = 0;
#pragma unroll
            for (int k = i + 1; k < 8; ++k) l[i] += v[k] < v[i] ? 1u : 0u;
        }
    } else {
        uint64_t s0, s1, s2;
#define DMS_OPERANDS                                                                                                \
    : [l0] "=&v"(l[0]), [l1] "=&v"(l[1]), [l2] "=&v"(l[2]), [l3] "=&v"(l[3]), [l4] "=&v"(l[4]), [l5] "=&v"(l[5]),     \
      [l6] "=&v"(l[6]), [s0] "=&s"(s0), [s1] "=&s"(s1), [s2] "=&s"(s2)                                              \
    : [v0] "v"(v[0]), [v1] "v"(v[1]), [v2] "v"(v[2]), [v3] "v"(v[3]), [v4] "v"(v[4]), [v5] "v"(v[5]), [v6] "v"(v[6]), \
      [v7] "v"(v[7])                                                                                                \
    : "vcc"
        if constexpr (sizeof(C) == 4) asm(DMS_DIGITS("i32") DMS_OPERANDS);
        else asm(DMS_DIGITS("f64") DMS_OPERANDS);
#undef DMS_OPERANDS
    }
}

// Batcher's odd-even merge sort of 16 inputs, without the comparators that
// touch the last two (which would hold the largest values): 53 comparators.
struct Comparators {
    uint8_t lo[64], hi[64];
    int n;
};

constexpr Comparators make_comparators(int inputs)
{
    Comparators N{};
    for (int p = 1; p < 16; p *= 2)
        for (int k = p; k >= 1; k /= 2)
            for (int j = k % p; j + k < 16; j += 2 * k)
                for (int i = 0; i < k; ++i)
                    if ((i + j) / (2 * p) == (i + j + k) / (2 * p) && i + j + k < inputs) {
                        N.lo[N.n] = (uint8_t)(i + j);
                        N.hi[N.n++] = (uint8_t)(i + j + k);
                    }
    return N;
}

constexpr Comparators kSort14 = make_comparators(14);
static_assert(kSort14.n == 53, "comparators of 14 inputs");

// The 14 neighbours in increasing order, 4 bits each; neighbours outside the
// grid compare above all others.  Ranks and single-precision values are sorted
// as doubles that carry the neighbour in their low bits, a minimum and a
// maximum per comparator (about 180 instructions; counting each neighbour's
// predecessors over the 91 pairs takes 330).  Double-precision values have no
// room for it and are counted.
template <typename Keys>
__device__ __forceinline__ uint64_t sorted_neighbours(const typename Keys::C *o)
{
    uint64_t at = 0;
    if constexpr (sizeof(typename Keys::C) <= 8) {
        double p[14];
#pragma unroll
        for (int e = 0; e < 14; ++e) p[e] = Keys::sort_key(o[e], e);
#pragma unroll
        for (int c = 0; c < kSort14.n; ++c) {
            const double a = p[kSort14.lo[c]], b = p[kSort14.hi[c]];
            p[kSort14.lo[c]] = min_packed(a, b);
            p[kSort14.hi[c]] = max_packed(a, b);
        }
        uint32_t w[2] = {0, 0};
#pragma unroll
        for (int r = 0; r < 14; ++r)
            w[r / 8] |= ((uint32_t)__double_as_longlong(p[r]) & 15u) << (4 * (r % 8));
        at = (uint64_t)w[1] << 32 | w[0];
        if constexpr (Keys::kSlots) at -= (at >> 3) & 0x1111111111111111ull;  // slot 8..14 is neighbour 7..13
    } else {
        uint32_t r[14];
#pragma unroll
        for (int e = 0; e < 14; ++e) r[e] = (uint32_t)e;
#pragma unroll
        for (int a = 0; a < 14; ++a)
#pragma unroll
            for (int b = a + 1; b < 14; ++b) {
                const uint32_t c = o[b] < o[a] ? 1u : 0u;
                r[a] += c;
                r[b] -= c;
            }
#pragma unroll
        for (int e = 1; e < 14; ++e) at |= (uint64_t)e << (4 * r[e]);
    }
    return at;
}

// The triangle of S with the smallest (kLargest: largest) key, as a one-bit
// set (S when it has at most one): walked from the highest rank down, keeping
// the triangles without (with) the neighbour of that rank when there are any.
// has[b] = triangle bits containing the neighbour of rank b.  A rank above the
// lower neighbours changes nothing, S holding lower triangles only, so the
// walk is straight-line code over all ranks but d's.
__device__ __forceinline__ uint32_t smallest_triangle(uint32_t S, const uint32_t *has)
{
#pragma unroll
    for (int b = 13; b >= 1; --b) {
        const uint32_t z = S & ~has[b];
        S = z ? z : S;
    }
    return S;
}

// Robins' pairing of the lower star of x, from its neighbours in increasing
// order (sorted_neighbours) and the mask of the lower ones.  Returns whether
// some cell of L(x) ends critical.
//
// Call the lower neighbours nodes, the lower triangles links (each joins two
// nodes) and compare links by their cells' keys.  Robins' queues give:
//  1. Edges.  An edge is paired when its node is reached by the smallest link
//     that joins a reached node to an unreached one: Prim's growth, with
//     distinct weights, so the links used are the minimum spanning forest of
//     the lower link, and each node's edge is paired with the link towards the
//     root, the lowest node of its component.  The first root's edge is paired
//     with x; every other root's edge is critical (it is declared when no link
//     reaches a new node, as the smallest unpaired edge).  Pairs with tets do
//     not interfere: a tet's last unpaired triangle t always has both nodes
//     reached (were one missing, t or another triangle of the tet would join
//     a reached node to it, and come first, faces preceding cofaces).
//  2. Tets.  The other links are left over for the tets.  A tet with one
//     unpaired triangle takes it; in whatever order that is done the result
//     is the same, since a leaf pair changes only cells above it.  When no
//     such tet is left but unpaired tets are, the smallest left-over triangle
//     is critical (all edges are settled and no tet can run out of triangles,
//     see 3), and the stripping goes on.
//  3. The left-over triangles and the tets form a forest whose trees end in
//     triangles with a missing or upper second tet, except when every
//     neighbour is lower: then the tets form one closed tree, stripped from
//     its leaves by increasing key, and the largest tet remains critical.
// The growth starts from d, the lowest node, with the nodes linked to it: the
// link to d is the smallest one at each of them.  Only links that avoid d
// matter afterwards, which fit one word (StarTables).  A link joins a reached
// to an unreached node exactly when it lies on an odd number of reached ones:
// reaching a node flips its links.
//
// Bound by vector-instruction issue: 63 instructions per node reached beyond
// d's neighbours (39 of them the search), 22 per tet, 47 per critical
// triangle, about 200 once, beside sorted_neighbours.  A wave of
// white noise reaches 4.9 nodes and strips 8.3 tets (its longest lane, dealt
// by lower-neighbour count).  It replaced a loop over single pairs that kept
// 60-bit sets of the unpaired cells and searched all of them each time (about
// 150 instructions a pair, 14 pairs a wave): gradient of 96 fields, half of
// them noise, 22.7 -> 17.0 ms; of a noisy 512^3 mixture 5.0 -> 3.8 ms; from
// the values of a 643 x 511 x 386 one 4.7 -> 3.2 ms.
__device__ __forceinline__ bool solve_star(uint64_t nb_at, uint32_t low, const StarTables &T, uint4 &out)
{
    if (low == 0) {  // L(x) = {x}: x is critical
        out = make_uint4(0, 0, 0, 0);
        return true;
    }
    const uint32_t d = (uint32_t)nb_at & 15u;
    const uint32_t F = T.link[d] & low;  // lower neighbours linked to d
    const uint4 *row = (const uint4 *)T.tris[d];
    uint32_t upper, S = 0, utets = 0;
    uint32_t b1;  // unpaired triangles of each tet = 2 b1 + b0: one for d's tets, three for the others
    {
        const uint4 r0 = row[0], r1 = row[1], r2 = row[2], r3 = row[3];
        const uint32_t c[14] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w, r2.x, r2.y, r2.z, r2.w, r3.x, r3.y};
        upper = r3.z;
        b1 = ~r3.w;
#pragma unroll
        for (int e = 0; e < 14; ++e) {
            const uint32_t lm = (uint32_t)((int32_t)(low << (31 - e)) >> 31), fm = (uint32_t)((int32_t)(F << (31 - e)) >> 31);
            upper |= c[e] & ~lm;
            utets |= kTables.edge_tetmask[e] & ~lm;
            S ^= c[e] & fm;
        }
    }
    const uint32_t L = ~upper;  // lower triangles (without d's)
    S &= L;
    uint32_t U = ~utets & 0xffffffu;  // unpaired lower tets
    uint32_t b0 = ~0u;
    uint32_t has[14];
#pragma unroll
    for (int b = 1; b < 14; ++b) has[b] = T.tris[d][nib(nb_at, b)];
    uint32_t reached = F | 1u << d;
    uint64_t edges;  // the edge fields
    {
        const uint32_t n0 = T.nibbles[reached & 127u], n1 = T.nibbles[reached >> 7];
        edges = T.fan[d] & ((uint64_t)n1 << 28 | n0);
    }
    bool crit = false;
    uint32_t left = L;  // lower triangles paired with no edge
    // 1. edges; every pass of the outer loop after the first starts a component
    for (int comp = 0; comp < 14; ++comp) {
        for (int step = 0; step < 14 && S; ++step) {
            const uint32_t bit = smallest_triangle(S, has);
            const uint64_t tri = T.tri[d][__builtin_ctz(bit)];
            const uint32_t ends = (uint32_t)(tri >> 32), D = (uint32_t)tri & 0xffffffu;
            const uint32_t f = (reached >> (ends & 15u)) & 1u ? ends >> 8 : ends;
            const uint32_t e = f & 15u;
            left ^= bit;
            b1 ^= D & ~b0;
            b0 ^= D;
            edges |= (uint64_t)((f >> 4) & 15u) << (4 * e);
            reached |= 1u << e;
            S ^= T.tris[d][e] & L;
        }
        const uint32_t rest = low & ~reached;
        if (!rest) break;
        uint32_t e = 0;  // the lowest node not reached
#pragma unroll
        for (int b = 13; b >= 1; --b) {
            const uint32_t g = nib(nb_at, b);
            e = (rest >> g) & 1u ? g : e;
        }
        crit = true;
        edges |= 2ull << (4 * e);
        reached |= 1u << e;
        S ^= T.tris[d][e] & L;
    }
    // 3. every neighbour lower: the largest tet is critical
    if (low == 0x3fffu) {
        uint32_t Q = 0xffffffu;
#pragma unroll 1
        for (int b = 13; b >= 0; --b) {
            const uint32_t z = Q & T.tris[nib(nb_at, b)][15];
            Q = z ? z : Q;
        }
        U &= ~Q;
        crit = true;
    }
    // 2. tets
    uint32_t ty = 0, tz = 0, tw = 0;  // the triangle fields, from the record's second word on
    for (int turn = 0; turn < 36 && U; ++turn) {
        uint32_t one = U & b0 & ~b1;
        for (int step = 0; step < 24 && one; ++step) {
            const uint32_t q = (uint32_t)__builtin_ctz(one);
            const uint64_t tet = T.tet[d][q];
            const uint32_t u = (uint32_t)tet & left;  // its one unpaired triangle
            const uint32_t tri = (uint32_t)T.tri[d][__builtin_ctz(u)], D = tri & 0xffffffu;
            const uint32_t second = u & (uint32_t)(tet >> 32) ? 0u : 1u;
            const uint4 w = *(const uint4 *)T.field[2u * (tri >> 24) + second];
            left ^= u;
            U &= ~(1u << q);
            b1 ^= D & ~b0;
            b0 ^= D;
            ty |= w.x;
            tz |= w.y;
            tw |= w.z;
            one = U & b0 & ~b1;
        }
        if (!U || !left) break;
        const uint32_t bit = smallest_triangle(left, has);
        const uint32_t D = (uint32_t)T.tri[d][__builtin_ctz(bit)] & 0xffffffu;
        left ^= bit;
        b1 ^= D & ~b0;
        b0 ^= D;
        crit = true;
    }
    out = make_uint4((uint32_t)edges, (uint32_t)(edges >> 32) | ty, tz, tw);
    return crit || left != 0;
}

// From the orders of x and its neighbours.
template <typename Keys>
__device__ __forceinline__ bool process_vertex(const typename Keys::C *o, typename Keys::C ox, const StarTables &T,
                                               uint4 &out)
{
    return solve_star(sorted_neighbours<Keys>(o), lower_mask(o, ox), T, out);
}

// ---------------------------------------------------------------------------
// Antipodal-regular vertices.  Neighbour e and neighbour 13 - e are opposite
// offsets.  When exactly one of each of the 7 opposite pairs precedes x (the
// common case of a smooth field: the lower link is a hemisphere), L(x) is
// fixed by which member of each pair is lower (7 bits) and by the order of
// those 7 neighbours (a permutation of 7).  Robins' result for all 128 x 5040
// such configurations is computed once per device by process_vertex itself
// and kept in a device table; such vertices then cost a table lookup.
constexpr int kPerm7 = 5040;
constexpr int kRegular = 128 * kPerm7;

// One-defect vertices: six pairs have one lower member and the seventh has
// both (8 lower neighbours) or neither (6).  All three families are looked
// up from one set of eight slots: v[i] = the member of pair i on the lower
// side (neighbour 13 - i when side bit i is set, else i) for i < 7, and
// v[7] = the smallest order among the other members -- neighbour j itself
// when pair j is wholly lower, else an upper order (replaced by a value
// above every order).  The Lehmer digits l_i count the later slots holding
// smaller orders; the codes are fixed-radix factorial sums of them:
//   code7 = sum over i < 7 of l_i (6 - i)!   (regular and |L| = 6)
//   code8 = sum over i < 8 of l_i (7 - i)!   (|L| = 8)
// For |L| = 6 slot j holds an upper order, larger than every lower one, so
// its digit is always 6 - j: the code is injective but sparse (one code in
// seven is used), which keeps the lookup free of any per-lane dependence on
// j beyond the table offset.
//   regular: index side * 7! + code7                       (10 MB)
//   |L| = 6: index (j * 64 + side6) * 7! + code7            (36 MB, sparse)
//   |L| = 8: index (j * 64 + side6) * 8! + code8            (289 MB)
// side6 is the 7-bit side pattern with bit j removed.  The three follow each
// other in one allocation per device, so that a lookup is one 32-bit entry
// number from one base; after the entries come the flags, one bit per entry:
// whether its lower star holds a critical cell.
constexpr int kPerm8 = 40320;
constexpr int kDefect6 = 7 * 64 * kPerm7;
constexpr int kDefect8 = 7 * 64 * kPerm8;
constexpr uint32_t kFirst6 = kRegular, kFirst8 = kFirst6 + kDefect6, kEntries = kFirst8 + kDefect8;
static_assert(kFirst6 % 64 == 0 && kFirst8 % 64 == 0 && kEntries % 64 == 0, "flag words per wave");
static_assert((uint64_t)kEntries * sizeof(uint4) < (1ull << 32), "32-bit byte offsets");
constexpr size_t kTableBytes = (size_t)kEntries * sizeof(uint4) + kEntries / 8;

__device__ __forceinline__ const uint32_t *table_flags(const uint4 *table)
{
    return (const uint32_t *)(table + kEntries);
}

// Whether x, with lower neighbours low, is in none of the tabulated families
// (at least two of the opposite pairs wholly lower or wholly upper).
__device__ __forceinline__ bool general_vertex(uint32_t low)
{
    return __popc((low ^ (__brev(low) >> 18)) & 0x7fu) < 6;
}

// m ? a : b for a mask m of all ones or all zeros.
__device__ __forceinline__ int32_t pick(uint32_t m, int32_t a, int32_t b)
{
    return (int32_t)(((uint32_t)a & m) | ((uint32_t)b & ~m));
}
__device__ __forceinline__ double pick(uint32_t m, double a, double b) { return m ? a : b; }
__device__ __forceinline__ unsigned __int128 pick(uint32_t m, unsigned __int128 a, unsigned __int128 b)
{
    return m ? a : b;
}

// Table entry of x (not a general vertex).
template <typename C>
__device__ __forceinline__ uint32_t table_entry(uint32_t low, const C *o)
{
    const C kHigh = c_highest<C>();
    const uint32_t rev = __brev(low) >> 18;  // bit e -> bit 13 - e
    const uint32_t one = (low ^ rev) & 0x7fu;
    const uint32_t side = __brev((low >> 7) & 0x7fu) >> 25;  // bit i: the lower member is 13 - i
    const uint32_t both = low & rev & 0x7fu;                   // pairs wholly lower
    // slot values without selecting between array elements by a per-lane
    // index (which the compiler expands into chains of compares): the lower
    // member of a single pair is the smaller order of the two; a wholly lower
    // pair (side bit set) takes neighbour 13 - i, and neighbour i goes to
    // slot 7
    C v[8];
    v[7] = kHigh;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const C a = o[i], b = o[13 - i];
        const uint32_t w = (uint32_t)__builtin_amdgcn_sbfe((int)both, i, 1);  // all ones or zeros
        v[i] = pick(w, b, cmin(a, b));
        v[7] = cmin(v[7], pick(w, a, kHigh));
    }
    uint32_t l[7];
    lehmer_digits(v, l);
    // factorial sums of the digits, by Horner's rule (in 24-bit products: the
    // full 32-bit multiply-add is four times slower)
    uint32_t code7 = l[0], code8 = l[0];
#pragma unroll
    for (int i = 1; i < 7; ++i) {
        code7 = __umul24(code7, (uint32_t)(7 - i)) + l[i];
        code8 = __umul24(code8, (uint32_t)(8 - i)) + l[i];
    }
    const bool eight = both != 0, regular = one == 0x7fu;
    const uint32_t j = (uint32_t)__builtin_ctz(~one | 0x80u);  // (7 for a regular vertex)
    const uint32_t side6 = (side & ((1u << j) - 1u)) | ((side >> (j + 1u)) << j);
    const uint32_t group = regular ? side : j * 64u + side6;
    const uint32_t first = eight ? kFirst8 : regular ? 0u : kFirst6;
    return __umul24(group, eight ? (uint32_t)kPerm8 : (uint32_t)kPerm7) + (eight ? code8 : code7) + first;
}

// Stores a row's record past the L2's ordinary replacement: a tile's 16 KB of
// records are not read again here, the halo planes it shares with the tiles
// above are.  (A 1026^3 gradient, 17 GB of records: 11.3 ms with ordinary
// stores, 10.2 ms so; 512^3: 3.52 and 3.50.)
__device__ __forceinline__ void store_record(uint4 *p, uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(u32x4{x, y, z, w}, (u32x4 *)p);
}

template <int GX, int GY>
struct Tile {
    static_assert(GX * GY == kTileVerts, "tile holds kTileVerts vertices");
    static constexpr int HX = GX + 2, HY = GY + 2, HZ = 3;
    static constexpr int kHalo = HX * HY * HZ;
};

// Comparison values of x's 14 neighbours (in neighbour order) and of x.
template <typename Keys, int GX, int GY>
__device__ __forceinline__ void gather_orders(const typename Keys::H *tile, int c, typename Keys::C *o,
                                              typename Keys::C &ox)
{
    using S = Tile<GX, GY>;
#pragma unroll
    for (int e = 0; e < 14; ++e)
        o[e] = Keys::cmp(tile[c + kTables.nb[e][0] + S::HX * (kTables.nb[e][1] + S::HY * kTables.nb[e][2])],
                         id_slot(e));
    ox = Keys::cmp(tile[c], 7);
}

// Vertices that no table covers ("general" vertices) are solved by solve_star,
// whose length varies with the lower star, so they leave the tile pass:
//  - a tile with few of them (the common case of a smooth field: one sparse
//    wave would hold the block's slot) sorts their neighbours while the halo
//    is in LDS and appends compact entries to a device queue, which
//    k_gradient_queue solves in full waves;
//  - a tile with kThreads of them or more is appended to a list of tiles,
//    which k_gradient_dense stages again and solves.
//   entry: x, y = sorted neighbours (56 bits), the record index (40 bits: z,
//          and the top byte of y), w = mask of the lower neighbours.
// Both are dealt to threads by the number of lower neighbours, which fixes
// most of the length (sorting by the number of steps itself would save 1%).
constexpr int kQueueChunk = 1024;  // entries per block of the queue kernel
constexpr int kSizeBins = 16;      // lower-neighbour counts (0..14)

__device__ __forceinline__ uint4 queue_entry(uint64_t nb_at, int64_t ridx, uint32_t low)
{
    const uint64_t r = (uint64_t)ridx;
    return make_uint4((uint32_t)nb_at, ((uint32_t)(nb_at >> 32) & 0x00ffffffu) | ((uint32_t)(r >> 32) << 24),
                      (uint32_t)r, low);
}
__device__ __forceinline__ uint64_t entry_neighbours(const uint4 &e)
{
    return (uint64_t)e.x | (uint64_t)(e.y & 0x00ffffffu) << 32;
}
__device__ __forceinline__ int64_t entry_record(const uint4 &e)
{
    return (int64_t)((uint64_t)e.z | (uint64_t)(e.y >> 24) << 32);
}

// The queue and the list of dense tiles, in the caller's workspace: a queue
// counter and a list counter, then the entries, then the tile numbers.  A
// counter may pass its capacity: entries beyond are not written (a launch has
// fewer than 2^24 tiles, its work items being a 32-bit number, and each adds less
// than kThreads to the queue's: it stays below 2^32).  A tile whose vertices do
// not all fit the queue solves the rest or is listed; when the list is full too
// the dense kernel takes every tile.  Without a workspace (all null) it does so
// in small launches; in others a tile with few vertices solves them itself, and
// a dense one marks one of its records.
struct Handoff {
    uint32_t *counts;  // [0] queue, [1] list
    uint4 *queue;
    uint32_t *list;
    uint32_t qcap, lcap;
};

__device__ __forceinline__ void load_tables(StarTables &T)
{
    const uint4 *src = (const uint4 *)&g_star;
    uint4 *dst = (uint4 *)&T;
    for (int i = threadIdx.x; i < (int)(sizeof(StarTables) / 16); i += kThreads) dst[i] = src[i];
}

// Exclusive scan of kSizeBins counters by the first wave.
__device__ __forceinline__ void scan_bins(uint32_t *bins)
{
    const int tid = threadIdx.x;
    if (tid < kWave) {
        const uint32_t v = tid < kSizeBins ? bins[tid] : 0u;
        uint32_t inc = v;
#pragma unroll
        for (int off = 1; off < kSizeBins; off <<= 1) {
            const uint32_t t = __shfl_up(inc, off);
            if (tid >= off) inc += t;
        }
        if (tid < kSizeBins) bins[tid] = inc - v;
    }
}

// First word of a dense tile's first record where there is no list: no record
// has it (edge fields end at 8).
constexpr uint32_t kDenseTile = 0xffffffffu;

// Marks record r (box index) as holding a critical cell: bit r of the mask.
__device__ __forceinline__ void mark_critical(uint32_t *mark, int64_t r)
{
    atomicOr(&mark[r >> 5], 1u << (uint32_t)(r & 31));
}

// A field's grid dims n, the owned box [lo, lo + w) and the index of its
// first record.
struct Box {
    int64_t n0, n1, n2, lo0, lo1, lo2, w0, w1, w2, rec_off;
};

// The thread's index, as a value that the compiler takes to be new at each
// call: what a tile's code derives from it is then not hoisted out of a loop
// over tiles (some 80 such values were, and spilled).
__device__ __forceinline__ int tile_thread()
{
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}

// Stages the comparison keys of tile (bx, by, bz) of the box, with a
// one-vertex halo, in LDS (no barrier afterwards).
template <typename Keys, int GX, int GY>
__device__ __forceinline__ void stage_halo(const void *__restrict__ field, const Box &B, int64_t bx, int64_t by,
                                           int64_t bz, int tid, uint32_t *flags, typename Keys::H *tile)
{
    using S = Tile<GX, GY>;
    const int64_t nx = B.n0, ny = B.n1, nz = B.n2;
    const int64_t x0 = B.lo0 + bx * GX - 1, y0 = B.lo1 + by * GY - 1, z0 = B.lo2 + bz - 1;
    const bool full = x0 >= 0 && y0 >= 0 && z0 >= 0 && x0 + S::HX <= nx && y0 + S::HY <= ny &&
                      z0 + S::HZ <= nz;
    bool nan = false, nan_any = false;
    bool staged = false;  // uniform
    if constexpr (GX == kWave) {
      using H = typename Keys::H;
      // inside the grid, and the tile's three planes within 32-bit byte
      // offsets of its first value
      if (full && (2 * nx * ny + S::HY * nx) * (int64_t)sizeof(H) < (1ll << 32)) {
        // rows of 66 values: wave w loads rows w, w + 4, ... (64 consecutive
        // values from a row address kept in scalar registers), and the first
        // 2 x 54 threads load the rows' last two values; every load is issued
        // before any LDS store.  A row's offset is its number times the row
        // stride, plus the rest of a plane for each plane before it; which
        // planes those are is known at compile time for all but one row.
        // (With each row's plane, line and 64-bit address computed from its
        // number the staging took 405 of the kernel's 670 scalar instructions
        // a wave.)
        constexpr int kRows = S::HY * S::HZ;
        constexpr int kWavesB = kThreads / kWave;
        constexpr int kPerRow = (kRows + kWavesB - 1) / kWavesB;
        static_assert(S::HX == kWave + 2 && 2 * kRows <= kThreads && kWavesB == 4 && S::HZ == 3, "row split");
        const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid / kWave) & 3u, lane = (uint32_t)tid % kWave;
        const char *first = (const char *)field + (x0 + nx * (y0 + ny * z0)) * (int64_t)sizeof(H);
        const uint32_t line = (uint32_t)nx * (uint32_t)sizeof(H);
        const uint32_t skip = (uint32_t)((ny - S::HY) * nx) * (uint32_t)sizeof(H);  // from a plane's rows to the next's
        H hv[kPerRow];
#pragma unroll
        for (int k = 0; k < kPerRow; ++k) {
            const uint32_t r = min(wave + (uint32_t)(kWavesB * k), (uint32_t)kRows - 1u);
            const char *row = first + (r * line + (r >= S::HY ? skip : 0u) + (r >= 2 * S::HY ? skip : 0u));
            hv[k] = Keys::load(row, lane, nan);
            nan_any |= nan;
        }
        const uint32_t er = tid < 2 * kRows ? (uint32_t)tid >> 1 : 0u;
        const uint32_t eo = er * line + (er >= S::HY ? skip : 0u) + (er >= 2 * S::HY ? skip : 0u);
        const H ev = Keys::load(first + eo, kWave + (tid & 1), nan);
        nan_any |= nan;
#pragma unroll
        for (int k = 0; k < kPerRow; ++k) {
            const uint32_t r = wave + (uint32_t)(kWavesB * k);
            if (r < (uint32_t)kRows) tile[r * S::HX + lane] = hv[k];
        }
        if (tid < 2 * kRows) tile[er * S::HX + kWave + (tid & 1)] = ev;
        staged = true;
      }
    }
    if (staged) {
    } else if (full && nx * S::HY < (1ll << 31)) {
        // inside the grid: each thread issues a fixed number of loads (its
        // last one clamped into the halo) before any LDS store, so that all
        // are in flight at once; a 64-bit base per halo plane and a 32-bit
        // offset within the plane
        static_assert(S::HZ == 3, "three halo planes");
        constexpr int kPlane = S::HX * S::HY;
        constexpr int kPer = (S::kHalo + kThreads - 1) / kThreads;
        const int nxi = (int)nx;
        const int64_t base0 = x0 + nx * (y0 + ny * z0), pstride = nx * ny;
        typename Keys::H hv[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = min(tid + j * kThreads, S::kHalo - 1);
            const int hz = i / kPlane, r = i - hz * kPlane;
            const int hy = r / S::HX, hx = r - hy * S::HX;
            const int64_t pb = hz == 0 ? base0 : (hz == 1 ? base0 + pstride : base0 + 2 * pstride);
            hv[j] = Keys::load(field, pb + hx + hy * nxi, nan);
            nan_any |= nan;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = tid + j * kThreads;
            if (i < S::kHalo) tile[i] = hv[j];
        }
    } else {
        for (int i = tid; i < S::kHalo; i += kThreads) {
            const int hx = i % S::HX, hy = (i / S::HX) % S::HY, hz = i / (S::HX * S::HY);
            const int64_t x = x0 + hx, y = y0 + hy, z = z0 + hz;
            typename Keys::H v = Keys::kAbsentH;
            if (x >= 0 && y >= 0 && z >= 0 && x < nx && y < ny && z < nz) {
                v = Keys::load(field, x + nx * (y + ny * z), nan);
                nan_any |= nan;
            }
            tile[i] = v;
        }
    }
    if (flags && __ballot(nan_any) && lane_id() == 0) atomicOr(flags, (uint32_t)DMS_FLAG_NAN);
}

// A wave whose first row of the tile is mostly general vertices (a noisy
// field) leaves all its vertices to the general path: the table index costs
// every lane of a row that has one.  in, gen: whether this lane's vertex of
// the first row lies in the box, and is general.
__device__ __forceinline__ bool skip_tables(bool in, bool gen)
{
    const int n = __popcll(__ballot(in)), g = __popcll(__ballot(in && gen));
    return g >= 32 && 2 * g > n;
}

// The table vertices of one GX x GY x 1 tile (1024 vertices, 4 per thread) of
// a box: their records from the precomputed tables.  The other vertices are
// handed over (Handoff).  tile_no: the tile's number in the launch.  Must be
// entered by the whole block.
//
// Bound by the record stores (16 B a vertex; a copy of the kernel without
// them takes half the time, one without table and flag reads five sixths),
// then by the latency of staging, table read and store one after the other:
// the vector work alone is a quarter.  So the three table families lie behind
// one 32-bit entry number (no branch or pointer per family), masks and digits
// are built from borrow and carry bits, and a row's loads have scalar
// addresses.  With a pointer, a branch and a loop per family, 1026^3 / 512^3 of
// ranks took 11.6 / 5.0 ms with the general vertices' kernels; so, with the
// records stored past the L2 and the tiles in chunks, 9.9 / 3.5 ms.
//
// The queue has room for one vertex in 16.  Fields with short sides have more
// general vertices (all of the boundary), and fill it.  The rest of a tile is
// then solved in its block while its neighbours are sorted and at hand; listed
// with the dense tiles, it is staged and searched again: 20 x 300 x 300 smooth
// ranks took 171 us so, now 98, a batch of 1000 smooth fields with sides 20..40
// 3.26 ms, now 2.40.  A launch of up to kListTiles tiles lists them: the dense
// kernel runs beside an idle chip there, and spreads a tile over four blocks (12
// fields, 758 tiles: 174 us of kernels, 180 when solved in the tile; 1200 tiles
// of 40 x 40 x 400: 65 and 61 us).
constexpr uint32_t kListTiles = 1024;

// Without a workspace, a launch of up to this many tiles leaves all general
// vertices to the dense kernel, a larger one marks its dense tiles.  Smooth and
// noise ranks, smooth values in double precision, us: 2048 tiles 58 / 97 / 116
// and, marked, 56 / 104 / 122; 3072 tiles 77 / 148 / 170 and 67 / 153 / 137; 8192
// tiles 194 / 370 / 410 and 116 / 374 / 263.
constexpr uint32_t kMarkTiles = 2048;

struct TileShared {
    uint32_t qbase, nlist;
    uint16_t list[kTileVerts];  // general vertices of the tile (tile positions)
};

template <typename Keys, int GX, int GY>
__device__ __forceinline__ void gradient_tile(const void *__restrict__ field, const Box &B, int64_t bx, int64_t by,
                                              int64_t bz, uint32_t tile_no, uint4 *__restrict__ rec,
                                              const uint4 *__restrict__ table, const Handoff &H, uint32_t *flags,
                                              uint32_t *__restrict__ mark, TileShared &sh,
                                              typename Keys::H *tile)
{
    using S = Tile<GX, GY>;
    using C = typename Keys::C;
    const int tid = threadIdx.x;
    const int64_t w0 = B.w0, w1 = B.w1, w2 = B.w2;
    if (tid == 0) sh.nlist = 0;
    stage_halo<Keys, GX, GY>(field, B, bx, by, bz, tid, flags, tile);
    __syncthreads();

    const int64_t rbase = B.rec_off + (bx * GX) + w0 * ((by * GY) + w1 * bz);
    // a 64-wide tile: vertex k of a thread lies in column lane and row
    // wave + 4 k, the same row for the whole wave, so the row's part of the
    // LDS and record addresses stays in scalar registers
    const int wave_u = __builtin_amdgcn_readfirstlane(tid / kWave);
    // all of a thread's table reads are issued (a vertex with no entry reads
    // a dummy one) before any record is stored, so that their latencies
    // overlap instead of adding up
    constexpr int kPer = kTileVerts / kThreads;
    uint32_t gx[kPer], gy[kPer], gz[kPer], gw[kPer];  // the entries, as plain words
    uint32_t fw[kPer];   // the flag words of the entries
    uint32_t fbit = 0;   // 5 bits per vertex: the entry's bit in its flag word
    uint32_t state = 0;  // bit k: vertex k in the box; bit kPer + k: it has an entry
    bool skip = false;   // uniform in the wave
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int v = tid + k * kThreads;
        const int tx = GX == kWave ? tid % kWave : v % GX;
        const int ty = GX == kWave ? wave_u + (kThreads / kWave) * k : v / GX;
        const bool in = bx * GX + tx < w0 && by * GY + ty < w1;
        uint32_t idx = 0;
        if (in) state |= 1u << k;
        if (!skip) {
            C o[14], ox;
            gather_orders<Keys, GX, GY>(tile, (tx + 1) + S::HX * ((ty + 1) + S::HY), o, ox);
            const uint32_t low = lower_mask(o, ox);
            const bool gen = general_vertex(low);
            if (k == 0) skip = skip_tables(in, gen);
            if (in && !gen && !skip) {
                idx = table_entry(low, o);
                state |= 1u << (kPer + k);
            }
        }
        const uint4 e = table[idx];
        gx[k] = e.x;
        gy[k] = e.y;
        gz[k] = e.z;
        gw[k] = e.w;
        fw[k] = table_flags(table)[idx >> 5];
        fbit |= (idx & 31u) << (5 * k);
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (!((state >> k) & 1u)) continue;
        const int v = tid + k * kThreads;
        const int tx = GX == kWave ? tid % kWave : v % GX;
        const int ty = GX == kWave ? wave_u + (kThreads / kWave) * k : v / GX;
        if ((state >> (kPer + k)) & 1u) {
            const int64_t r = rbase + tx + w0 * ty;
            store_record(rec + r, gx[k], gy[k], gz[k], gw[k]);
            if (mark && ((fw[k] >> ((fbit >> (5 * k)) & 31u)) & 1u)) mark_critical(mark, r);
        } else {
            sh.list[atomicAdd(&sh.nlist, 1u)] = (uint16_t)v;
        }
    }
    __syncthreads();
    const uint32_t total = sh.nlist;
    if (total == 0) return;

    const Handoff Q = H;
    bool dense = total >= (uint32_t)kThreads;
    if (!Q.counts) {
        if (gridDim.x <= kMarkTiles) return;
        if (dense) {
            // (by the thread that stored the table entry there, if it has one)
            if (tid == 0) store_record(rec + rbase, kDenseTile, kDenseTile, kDenseTile, kDenseTile);
            return;
        }
    }
    if (!dense) {
        // reserve queue slots; the sorting below overlaps the atomic
        if (tid == 0) sh.qbase = Q.counts ? atomicAdd(&Q.counts[0], total) : 0u;
        const bool mine = (uint32_t)tid < total;
        const int v = mine ? sh.list[tid] : 0;
        const int tx = v % GX, ty = v / GX;
        const int c = (tx + 1) + S::HX * ((ty + 1) + S::HY);
        uint32_t low = 0;
        uint64_t nb_at = 0;
        if (mine) {
            C o[14], ox;
            gather_orders<Keys, GX, GY>(tile, c, o, ox);
            low = lower_mask(o, ox);
            nb_at = sorted_neighbours<Keys>(o);
        }
        __syncthreads();
        // as many as fit are queued, so that every slot the queue kernel
        // reads, [0, min(count, qcap)), has been written by this launch
        const int64_t ridx = rbase + tx + w0 * ty;
        const uint32_t qb = sh.qbase;
        const uint32_t nq = qb >= Q.qcap ? 0u : min(total, Q.qcap - qb);  // uniform
        if ((uint32_t)tid < nq) Q.queue[qb + tid] = queue_entry(nb_at, ridx, low);
        if (nq == total) return;
        if (gridDim.x > kListTiles || !Q.counts) {
            // solved here, with the tables in place of the halo
            static_assert(sizeof(StarTables) <= sizeof(typename Keys::H) * S::kHalo, "tables in the halo's space");
            StarTables &T = *(StarTables *)tile;
            load_tables(T);
            __syncthreads();
            if (mine && (uint32_t)tid >= nq) {
                uint4 r;
                const bool crit = solve_star(nb_at, low, T, r);
                rec[ridx] = r;
                if (mark && crit) mark_critical(mark, ridx);
            }
            return;
        }
        dense = true;  // listed too: the dense kernel solves all of the tile's general vertices
    }
    if (dense && tid == 0) {
        const uint32_t at = atomicAdd(&Q.counts[1], 1u);
        if (at < Q.lcap) Q.list[at] = tile_no;
    }
}

// Column order: tile t of a box of bxc x (any) x nz tiles, in 32-bit divisions
// (a launch has fewer than 2^31 tiles, a side fewer than 2^31 vertices).
struct TileAt {
    uint32_t x, y, z;
};

__device__ __forceinline__ TileAt tile_at(uint32_t t, uint32_t nz, uint32_t bxc)
{
    const uint32_t col = t / nz, by = col / bxc;
    return TileAt{col - by * bxc, by, t - col * nz};
}

// Tile taken by block b of `blocks`: blocks go to the XCDs in turn, so that
// every eighth block of a group of 64 shares an L2; these take eight tiles in
// a row, each of which reads two of the last one's three halo planes.
// (Chunks of 8 / 32 / 512 tiles: 9.91 / 9.92 / 10.02 ms for 1026^3 ranks, 3.45
// / 3.45 / 3.46 for 512^3; tiles in block order 10.18 and 3.50.)
constexpr uint32_t kChunk = 8;

__device__ __forceinline__ uint32_t chunked_tile(uint32_t b, uint32_t blocks)
{
    constexpr uint32_t kXcds = 8, kGroup = kXcds * kChunk;
    const uint32_t g = b / kGroup;
    if ((g + 1) * kGroup > blocks) return b;
    const uint32_t r = b - g * kGroup;
    return g * kGroup + (r % kXcds) * kChunk + r / kXcds;
}

// Keys: RankKeys reads the int32 order; F32Keys / F64Keys read the values
// (flags receives DMS_FLAG_NAN for a NaN among them).
// Tiles in column order, z fastest: the tiles running at the same time then
// include each tile's neighbours above and below, which read two of its
// three halo planes, so most halo reads hit a cache (row order, with z
// slowest, put those neighbours a whole plane of tiles apart).
template <typename Keys, int GX, int GY>
__global__ __launch_bounds__(kThreads, 8) void k_gradient(const void *__restrict__ field, Box B, uint32_t bx_count,
                                                          uint4 *__restrict__ rec,
                                                          const uint4 *__restrict__ table, Handoff H,
                                                          uint32_t *flags, uint32_t *__restrict__ mark)
{
    __shared__ TileShared sh;
    __shared__ __align__(16) typename Keys::H tile[Tile<GX, GY>::kHalo];
    const uint32_t t = chunked_tile(blockIdx.x, gridDim.x);
    const TileAt T = tile_at(t, (uint32_t)B.w2, bx_count);
    const int64_t bx = T.x, by = T.y, bz = T.z;
    gradient_tile<Keys, GX, GY>(field, B, bx, by, bz, t, rec, table, H, flags, mark, sh, tile);
}

// Batched form: many whole fields, concatenated; one block per tile of the
// (field, tile) list, field f owning tiles [tile_start[f], tile_start[f+1]).
// tile_field[t] names the field of tile t, so a block finds its field with
// one read, and the kernel keeps the single-field kernel's registers and LDS
// (a persistent grid walking the tiles held the walk's 64-bit state in
// scalar registers and spilled).
struct BatchTiles {
    const BatchField *fields;
    const int64_t *tile_start;
    const uint16_t *tile_field;
};

template <int GX, int GY>
__device__ __forceinline__ Box batch_box(const BatchTiles &L, int64_t t, int64_t &bx, int64_t &by, int64_t &bz)
{
    const int f = L.tile_field[t];
    const BatchField F = L.fields[f];
    // column order inside the field, as in k_gradient
    const TileAt T = tile_at((uint32_t)(t - L.tile_start[f]), (uint32_t)F.n[2], (uint32_t)((F.n[0] + GX - 1) / GX));
    bx = T.x;
    by = T.y;
    bz = T.z;
    return Box{F.n[0], F.n[1], F.n[2], 0, 0, 0, F.n[0], F.n[1], F.n[2], F.off};
}

template <int GX, int GY>
__global__ __launch_bounds__(kThreads, 8) void k_gradient_batch(const int32_t *__restrict__ order, BatchTiles L,
                                                                uint4 *__restrict__ rec,
                                                                const uint4 *__restrict__ table, Handoff H,
                                                                uint32_t *__restrict__ mark)
{
    __shared__ TileShared sh;
    __shared__ __align__(16) int32_t tile[Tile<GX, GY>::kHalo];
    int64_t bx, by, bz;
    const uint32_t t = chunked_tile(blockIdx.x, gridDim.x);
    const Box B = batch_box<GX, GY>(L, t, bx, by, bz);
    gradient_tile<RankKeys, GX, GY>(order + B.rec_off, B, bx, by, bz, t, rec, table, H, nullptr, mark, sh,
                                    tile);
}

// All vertices of one tile that gradient_tile left (whole: all of its
// vertices), solved in rounds of kThreads, dealt by the number of lower
// neighbours.  part of parts (1 or 4): the quarter of the tile's positions
// this block takes.  first: position 0 is solved in any case (its record holds
// the tile's mark).
struct DenseShared {
    StarTables T;
    uint32_t bins[kSizeBins];
    uint32_t crit[kTileVerts / 32];  // bit v: tile position v holds a critical cell
    uint16_t perm[kTileVerts];       // tile positions by lower-neighbour count
};

template <typename Keys, int GX, int GY>
__device__ __forceinline__ void dense_tile(const void *__restrict__ field, const Box &B, int64_t bx, int64_t by,
                                           int64_t bz, int part, int parts, bool whole, bool first,
                                           uint4 *__restrict__ rec, uint32_t *flags, uint32_t *__restrict__ mark,
                                           DenseShared &sh, typename Keys::H *tile)
{
    using S = Tile<GX, GY>;
    using C = typename Keys::C;
    constexpr int kPer = kTileVerts / kThreads;
    const int tid = tile_thread();
    stage_halo<Keys, GX, GY>(field, B, bx, by, bz, tid, flags, tile);
    if (tid < kSizeBins) sh.bins[tid] = 0;
    if (tid < kTileVerts / 32) sh.crit[tid] = 0;
    __syncthreads();
    uint32_t sizes = 0;  // 8 bits per vertex: lower-neighbour count, bit 7 set for a vertex to be solved
    bool skip = false;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int v = tid + k * kThreads;
        const bool mine = parts == 1 || k == part;  // uniform
        if (k > 0 && !mine) continue;
        const int tx = v % GX, ty = v / GX;
        const bool in = bx * GX + tx < B.w0 && by * GY + ty < B.w1;
        C o[14], ox;
        gather_orders<Keys, GX, GY>(tile, (tx + 1) + S::HX * ((ty + 1) + S::HY), o, ox);
        const uint32_t low = lower_mask(o, ox);
        const bool gen = general_vertex(low);
        if (k == 0) skip = skip_tables(in, gen);
        if (mine && in && (gen || whole || skip || (first && v == 0))) {
            const uint32_t m = (uint32_t)__popc(low);
            sizes |= (128u | m) << (8 * k);
            atomicAdd(&sh.bins[m], 1u);
        }
    }
    __syncthreads();
    scan_bins(sh.bins);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t s = (sizes >> (8 * k)) & 255u;
        if (s & 128u) sh.perm[atomicAdd(&sh.bins[s & 15u], 1u)] = (uint16_t)(tid + k * kThreads);
    }
    __syncthreads();
    const uint32_t total = sh.bins[kSizeBins - 1];  // its own bin is empty: the end of the last one
    const int64_t rbase = B.rec_off + (bx * GX) + B.w0 * ((by * GY) + B.w1 * bz);
    for (uint32_t base = 0; base < total; base += kThreads) {
        const uint32_t i = base + tid;
        if (i < total) {
            const int v = sh.perm[i];
            const int tx = v % GX, ty = v / GX;
            C o[14], ox;
            gather_orders<Keys, GX, GY>(tile, (tx + 1) + S::HX * ((ty + 1) + S::HY), o, ox);
            uint4 r;
            if (process_vertex<Keys>(o, ox, sh.T, r)) atomicOr(&sh.crit[v / 32], 1u << (v % 32));
            rec[rbase + tx + B.w0 * ty] = r;
        }
    }
    __syncthreads();
    // the mask bits of 16 positions of a row at a time
    if (mark && tid < kTileVerts / 16) {
        const uint64_t bits = (sh.crit[tid / 2] >> (16 * (tid % 2))) & 0xffffu;
        if (bits) {
            const int v = 16 * tid;
            const int64_t r = rbase + v % GX + B.w0 * (v / GX);
            const uint64_t m = bits << (r & 31);
            if ((uint32_t)m) atomicOr(&mark[r >> 5], (uint32_t)m);
            if (m >> 32) atomicOr(&mark[(r >> 5) + 1], (uint32_t)(m >> 32));
        }
    }
    __syncthreads();
}

// The listed tiles (every tile when there is no list or it overflowed), dealt
// to a grid of at most kDenseBlocks blocks.  A list with less than a quarter
// of a tile per block is dealt in quarter tiles, which repeat only the staging.
constexpr int kDenseBlocks = 256 * 6;
constexpr int64_t kWholeTiles = 256;  // launches of at most this many tiles use the dense kernel alone

template <typename Solve>
__device__ __forceinline__ void dense_walk(const Handoff &H, uint32_t ntiles, Solve solve)
{
    uint32_t n = ntiles;
    const uint32_t *list = nullptr;
    if (H.counts && H.counts[1] <= H.lcap) {
        n = H.counts[1];
        list = H.list;
    }
    const int parts = (uint64_t)n * 4 <= gridDim.x ? 4 : 1;
    for (uint64_t i = blockIdx.x; i < (uint64_t)n * parts; i += gridDim.x) {
        const uint32_t j = (uint32_t)(i / parts);
        solve(list ? list[j] : j, (int)(i % parts), parts);
    }
}

// whole (without a list): the kernel does all vertices of all tiles by itself.
// With few tiles the time is the latency of one tile and of the launches, and
// a table lookup saves nothing: k_gradient, this kernel and the queue's took
// 13 + 18 + 20 us on a 24 x 20 x 16 noise field, this kernel alone 20.  At 256
// tiles (64^3) the whole call takes, smooth and noise, 20 and 27 us of ranks, 27
// and 36 of double-precision values; with tables and queue 44 and 37, 57 and 48.
template <typename Keys, int GX, int GY>
__global__ __launch_bounds__(kThreads, 6) void k_gradient_dense(const void *__restrict__ field, Box B,
                                                                uint32_t bx_count, uint32_t ntiles, bool whole,
                                                                uint4 *__restrict__ rec, Handoff H, uint32_t *flags,
                                                                uint32_t *__restrict__ mark)
{
    __shared__ DenseShared sh;
    __shared__ typename Keys::H tile[Tile<GX, GY>::kHalo];
    load_tables(sh.T);
    dense_walk(H, ntiles, [&](uint32_t t, int part, int parts) {
        const TileAt T = tile_at(t, (uint32_t)B.w2, bx_count);
        const int64_t bx = T.x, by = T.y, bz = T.z;
        dense_tile<Keys, GX, GY>(field, B, bx, by, bz, part, parts, whole, false, rec, flags, mark, sh, tile);
    });
}

// The same without a workspace: the tiles that are marked.  A block asks for
// kThreads of its tiles at once.  (With every tile staged and searched again the
// gradient of a smooth 256^3 field took 367 us, of a 512^3 one 2.34 ms; now 166 us
// and 1.05 ms.)
// Its tiles are kMarkedBlocks apart, a prime, or a block could get a column's
// bottom or top tile (all dense) every time: a smooth 256^3 field took 323 us with
// kDenseBlocks.
constexpr uint32_t kMarkedBlocks = 1531;
static_assert(kMarkedBlocks <= kMarkTiles, "fewer blocks than tiles");

template <typename Keys, int GX, int GY>
__global__ __launch_bounds__(kThreads, 6) void k_gradient_marked(const void *__restrict__ field, Box B,
                                                                 uint32_t bx_count, uint32_t ntiles,
                                                                 uint4 *__restrict__ rec,
                                                                 uint32_t *__restrict__ mark)
{
    __shared__ DenseShared sh;
    __shared__ uint64_t found[kThreads / kWave];
    __shared__ typename Keys::H tile[Tile<GX, GY>::kHalo];
    load_tables(sh.T);
    for (uint64_t t0 = blockIdx.x; t0 < ntiles; t0 += (uint64_t)gridDim.x * kThreads) {
        const uint64_t mine = t0 + (uint64_t)gridDim.x * threadIdx.x;
        bool marked = false;
        if (mine < ntiles) {
            const TileAt T = tile_at((uint32_t)mine, (uint32_t)B.w2, bx_count);
            marked = rec[(int64_t)T.x * GX + B.w0 * ((int64_t)T.y * GY + B.w1 * T.z)].x == kDenseTile;
        }
        const uint64_t bits = __ballot(marked);
        __syncthreads();
        if (lane_id() == 0) found[threadIdx.x / kWave] = bits;
        __syncthreads();
        for (int w = 0; w < kThreads / kWave; ++w)
            for (uint64_t left = found[w]; left; left &= left - 1u) {
                const uint64_t t = t0 + (uint64_t)gridDim.x * (uint32_t)(kWave * w + __builtin_ctzll(left));
                const TileAt T = tile_at((uint32_t)t, (uint32_t)B.w2, bx_count);
                const int64_t bx = T.x, by = T.y, bz = T.z;
                dense_tile<Keys, GX, GY>(field, B, bx, by, bz, 0, 1, false, true, rec, nullptr, mark, sh, tile);
            }
    }
}

template <int GX, int GY>
__global__ __launch_bounds__(kThreads, 6) void k_gradient_dense_batch(const int32_t *__restrict__ order, BatchTiles L,
                                                                      uint32_t ntiles, bool whole,
                                                                      uint4 *__restrict__ rec, Handoff H,
                                                                      uint32_t *__restrict__ mark)
{
    __shared__ DenseShared sh;
    __shared__ int32_t tile[Tile<GX, GY>::kHalo];
    load_tables(sh.T);
    dense_walk(H, ntiles, [&](uint32_t t, int part, int parts) {
        int64_t bx, by, bz;
        const Box B = batch_box<GX, GY>(L, t, bx, by, bz);
        dense_tile<RankKeys, GX, GY>(order + B.rec_off, B, bx, by, bz, part, parts, whole, false, rec, nullptr, mark,
                                     sh, tile);
    });
}

// Zeroes the mask and the handoff's two counters (either may be null).
__global__ void k_gradient_begin(uint32_t *__restrict__ mark, int64_t words, uint32_t *counts)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (mark && i < words) mark[i] = 0u;
    if (counts && i < 2) counts[i] = 0u;
}

// Solves the queued general vertices: block b takes a chunk of the filled
// part, sorts it by the number of lower neighbours and solves it in full
// rounds.  A short queue is cut into chunks of one round, for more blocks (a
// long one into kQueueChunk entries, whose waves are more even).
__global__ __launch_bounds__(kThreads, 8) void k_gradient_queue(const uint4 *__restrict__ queue,
                                                                const uint32_t *qcount, uint32_t qcap,
                                                                uint4 *__restrict__ rec,
                                                                uint32_t *__restrict__ mark)
{
    __shared__ StarTables T;
    __shared__ uint32_t bins[kSizeBins];
    __shared__ uint16_t perm[kQueueChunk];
    const int tid = threadIdx.x;
    const uint32_t filled = min(*qcount, qcap);
    const uint32_t chunk =
        filled <= 1024u * kThreads && (uint64_t)filled <= (uint64_t)gridDim.x * kThreads ? kThreads : kQueueChunk;
    const uint64_t start = (uint64_t)blockIdx.x * chunk;
    if (start >= filled) return;  // uniform
    const uint32_t cnt = (uint32_t)min<uint64_t>(chunk, filled - start);
    load_tables(T);
    if (tid < kSizeBins) bins[tid] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += kThreads) atomicAdd(&bins[__popc(queue[start + i].w) & 15], 1u);
    __syncthreads();
    scan_bins(bins);
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += kThreads)
        perm[atomicAdd(&bins[__popc(queue[start + i].w) & 15], 1u)] = (uint16_t)i;
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += kThreads) {
        const uint4 e = queue[start + perm[i]];
        uint4 r;
        const bool crit = solve_star(entry_neighbours(e), e.w & 0x3fffu, T, r);
        const int64_t ri = entry_record(e);
        rec[ri] = r;
        if (mark && crit) mark_critical(mark, ri);
    }
}

// Decodes a Lehmer code (factorial base, first item most significant) of
// N items into their ranks.
template <int N>
__device__ void lehmer_decode(uint32_t code, uint32_t *rank)
{
    uint32_t w = 1;
    for (int i = 2; i < N; ++i) w *= (uint32_t)i;  // (N - 1)!
    uint32_t used = 0;
    for (int i = 0; i < N; ++i) {
        uint32_t l = code / w;
        code %= w;
        if (i < N - 1) w /= (uint32_t)(N - 1 - i);
        int r = 0;  // the l-th smallest unused rank
        for (;; ++r)
            if (!((used >> r) & 1u)) {
                if (l == 0) break;
                --l;
            }
        used |= 1u << r;
        rank[i] = (uint32_t)r;
    }
}

// Fills the regular-vertex table: entry side * 5040 + code holds the record of
// the configuration whose lower neighbours are, for pair i, neighbour i or
// 13 - i (bit i of side), ordered by the permutation with Lehmer code `code`.
__global__ __launch_bounds__(kThreads) void k_regular_table(uint4 *__restrict__ table)
{
    __shared__ StarTables T;
    load_tables(T);
    __syncthreads();
    const int idx = blockIdx.x * kThreads + threadIdx.x;  // a wave covers 64 aligned entries
    bool crit = false;
    if (idx < kRegular) {
        const uint32_t side = idx / kPerm7;
        uint32_t rank[7];
        lehmer_decode<7>(idx % kPerm7, rank);
        int32_t o[14];
        for (int i = 0; i < 7; ++i) {
            const int lowm = ((side >> i) & 1u) ? 13 - i : i;
            o[lowm] = (int32_t)rank[i];
            o[13 - lowm] = 100 + i;  // above x
        }
        uint4 r;
        crit = process_vertex<RankKeys>(o, 50, T, r);
        table[idx] = r;
    }
    const uint64_t m = __ballot(crit);
    if (lane_id() == 0 && idx < kRegular) {
        uint32_t *flags = (uint32_t *)(table + kEntries);
        flags[idx / 32] = (uint32_t)m;
        flags[idx / 32 + 1] = (uint32_t)(m >> 32);
    }
}

// Fills a one-defect table in the layout table_entry reads: for |L| = 8 the
// code is that of 8 slots (slot 7 = neighbour j); for |L| = 6 that of 7
// slots where slot j (pair j, wholly upper) ranks above the other six --
// entries whose code puts it elsewhere are never read and stay zero.
template <bool kEight>
__global__ __launch_bounds__(kThreads) void k_defect_table(uint4 *__restrict__ table)
{
    __shared__ StarTables T;
    load_tables(T);
    __syncthreads();
    constexpr int N = kEight ? 8 : 7;
    constexpr int64_t perms = kEight ? kPerm8 : kPerm7;
    constexpr int64_t total = 7 * 64 * perms;
    constexpr uint32_t first = kEight ? kFirst8 : kFirst6;
    uint32_t *flags = (uint32_t *)(table + kEntries) + first / 32;
    const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;  // a wave covers 64 aligned entries
    bool crit = false;
    if (idx < total) {
        const uint32_t code = (uint32_t)(idx % perms);
        const uint32_t js = (uint32_t)(idx / perms);
        const uint32_t j = js / 64, side6 = js % 64;
        // the 7-bit side pattern with bit j (pair j) set for both lower
        const uint32_t side = (side6 & ((1u << j) - 1u)) | ((side6 >> j) << (j + 1u)) |
                              (kEight ? 1u << j : 0u);
        uint32_t rank[N];
        lehmer_decode<N>(code, rank);
        uint4 r = make_uint4(0, 0, 0, 0);
        if (kEight || rank[j] == 6u) {  // other |L| = 6 codes are never read
            int32_t o[14];
            for (int e = 0; e < 14; ++e) o[e] = 100 + e;  // above x unless set below
            for (int i = 0; i < 7; ++i) {
                if (!kEight && (uint32_t)i == j) continue;
                o[((side >> i) & 1u) ? 13 - i : i] = (int32_t)rank[i];
            }
            if (kEight) o[j] = (int32_t)rank[7];
            crit = process_vertex<RankKeys>(o, 50, T, r);
        }
        table[first + idx] = r;
    }
    const uint64_t m = __ballot(crit);
    if (lane_id() == 0 && idx < total) {
        flags[idx / 32] = (uint32_t)m;
        flags[idx / 32 + 1] = (uint32_t)(m >> 32);
    }
}

}  // namespace
}  // namespace dms

namespace dms {

namespace {
std::atomic<uint64_t> g_regular_ready{0};  // one bit per device that holds the tables
std::mutex g_table_mutex;
uint4 *g_table_ptr[64];  // per device, held until the process ends
}

int init_tables(hipStream_t s)
{
    if (const int dc = device_check()) return dc;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DMS_E_HIP;
    const uint64_t bit = 1ull << dev;
    if (g_regular_ready.load() & bit) return DMS_OK;
    std::lock_guard<std::mutex> lock(g_table_mutex);
    if (g_regular_ready.load() & bit) return DMS_OK;
    if (!g_table_ptr[dev]) {
        void *p = nullptr;
        if (hipMalloc(&p, kTableBytes) != hipSuccess) return DMS_E_HIP;
        g_table_ptr[dev] = (uint4 *)p;
    }
    uint4 *table = g_table_ptr[dev];
    hipLaunchKernelGGL(k_regular_table, dim3((kRegular + kThreads - 1) / kThreads), dim3(kThreads), 0, s, table);
    hipLaunchKernelGGL(k_defect_table<false>, dim3((kDefect6 + kThreads - 1) / kThreads), dim3(kThreads), 0, s, table);
    hipLaunchKernelGGL(k_defect_table<true>, dim3((kDefect8 + kThreads - 1) / kThreads), dim3(kThreads), 0, s, table);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return DMS_E_HIP;
    g_regular_ready.fetch_or(bit);
    return DMS_OK;
}

// The current device's tables (null before init_tables).
static const uint4 *device_tables()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    return (g_regular_ready.load() >> dev) & 1u ? g_table_ptr[dev] : nullptr;
}

// DMS_OK when the current device is a gfx950 whose tables init_tables has
// filled; DMS_E_UNSUPPORTED or DMS_E_NOT_INITIALISED otherwise.
int tables_ready()
{
    if (const int dc = device_check()) return dc;
    return device_tables() ? DMS_OK : DMS_E_NOT_INITIALISED;
}


// Workspace: 256 bytes of counters, then room for one vertex in 16 plus a
// chunk as 16-byte queue entries, of which the last 1/256 of a vertex each
// hold the list of dense tiles (4 bytes a tile).  A dense tile has at least
// kThreads vertices, so the list has room for all of them and for three times
// as many tiles that found the queue full.
static int64_t workspace_slots(int64_t owned)
{
    const int64_t c = owned / 16 + kQueueChunk;
    return c < 0x7fffffffLL ? c : 0x7fffffffLL;
}

size_t gradient_workspace_size(int64_t owned) { return 256 + (size_t)workspace_slots(owned) * sizeof(uint4); }

// Carves the workspace (all null when ws is null).
static Handoff handoff_carve(char *ws, int64_t owned)
{
    Handoff H{nullptr, nullptr, nullptr, 0, 0};
    if (!ws) return H;
    const int64_t slots = workspace_slots(owned);
    int64_t lslots = owned / kThreads + 16;
    if (lslots > slots / 2) lslots = slots / 2;
    H.counts = (uint32_t *)ws;
    H.queue = (uint4 *)(ws + 256);
    H.qcap = (uint32_t)(slots - lslots);
    H.list = (uint32_t *)(H.queue + H.qcap);
    H.lcap = (uint32_t)(lslots < 0x1fffffff ? 4 * lslots : 0x7fffffff);
    return H;
}

// Clears the mask of `owned` records and the handoff's counters.
static void gradient_begin(uint32_t *mark, int64_t owned, const Handoff &H, hipStream_t s)
{
    if (!mark && !H.counts) return;
    const int64_t words = mark ? (owned + 31) / 32 : 2;
    hipLaunchKernelGGL(k_gradient_begin, dim3((unsigned)((words + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                       mark, words, H.counts);
}

static void queue_finish(const Handoff &H, uint32_t *rec, uint32_t *mark, hipStream_t s)
{
    if (!H.counts) return;
    const unsigned blocks = (unsigned)(((int64_t)H.qcap + kQueueChunk - 1) / kQueueChunk);
    hipLaunchKernelGGL(k_gradient_queue, dim3(blocks), dim3(kThreads), 0, s, H.queue, H.counts, H.qcap,
                       (uint4 *)rec, mark);
}

static unsigned dense_blocks(int64_t ntiles) { return (unsigned)(4 * ntiles < kDenseBlocks ? 4 * ntiles : kDenseBlocks); }

template <typename Keys>
static int launch_gradient_keys(const void *field, const int64_t *dims, const int64_t *lo,
                                const int64_t *hi, uint32_t *rec, uint32_t *mark, char *ws, uint32_t *flags,
                                hipStream_t s)
{
    const Box B{dims[0], dims[1], dims[2], lo[0], lo[1], lo[2], hi[0] - lo[0], hi[1] - lo[1], hi[2] - lo[2], 0};
    if (B.w0 == 0 || B.w1 == 0 || B.w2 == 0) return DMS_OK;
    const int64_t owned = B.w0 * B.w1 * B.w2;
    constexpr int kGX = kTileX[0], kGY = kTileVerts / kGX;
    const int64_t bxc = (B.w0 + kGX - 1) / kGX, byc = (B.w1 + kGY - 1) / kGY;
    const int64_t blocks = bxc * byc * B.w2;
    if (blocks > 2147483647LL) return DMS_E_SIZE;
    const bool whole = blocks <= kWholeTiles;
    const Handoff H = handoff_carve(whole ? nullptr : ws, owned);
    gradient_begin(mark, owned, H, s);
    if (!whole)
        hipLaunchKernelGGL((k_gradient<Keys, kGX, kGY>), dim3((unsigned)blocks), dim3(kThreads), 0, s, field, B, (uint32_t)bxc,
                           (uint4 *)rec, device_tables(), H, flags, mark);
    if (whole || H.counts || blocks <= (int64_t)kMarkTiles)
        hipLaunchKernelGGL((k_gradient_dense<Keys, kGX, kGY>), dim3(dense_blocks(blocks)), dim3(kThreads), 0, s, field,
                           B, (uint32_t)bxc, (uint32_t)blocks, whole, (uint4 *)rec, H, whole ? flags : nullptr, mark);
    else
        hipLaunchKernelGGL((k_gradient_marked<Keys, kGX, kGY>), dim3(kMarkedBlocks), dim3(kThreads), 0, s, field, B,
                           (uint32_t)bxc, (uint32_t)blocks, (uint4 *)rec, mark);
    queue_finish(H, rec, mark, s);
    return launch_status();
}

int launch_gradient_batch(int variant, const int32_t *order, const BatchField *fields, int nfields,
                          const int64_t *tile_start, const uint16_t *tile_field, int64_t total_tiles,
                          int64_t total_verts, uint32_t *rec, uint32_t *mark, char *ws, hipStream_t s)
{
    (void)nfields;
    if (total_tiles == 0) return DMS_OK;
    if (total_tiles > 2147483647LL) return DMS_E_SIZE;
    const uint4 *table = device_tables();
    const bool whole = total_tiles <= kWholeTiles;
    const Handoff H = handoff_carve(whole ? nullptr : ws, total_verts);
    gradient_begin(mark, total_verts, H, s);
    const BatchTiles L{fields, tile_start, tile_field};
#define DMS_LAUNCH(GXV)                                                                                             \
    if (!whole)                                                                                                      \
        hipLaunchKernelGGL((k_gradient_batch<GXV, kTileVerts / GXV>), dim3((unsigned)total_tiles), dim3(kThreads),   \
                           0, s, order, L, (uint4 *)rec, table, H, mark);                                               \
    hipLaunchKernelGGL((k_gradient_dense_batch<GXV, kTileVerts / GXV>), dim3(dense_blocks(total_tiles)),             \
                       dim3(kThreads), 0, s, order, L, (uint32_t)total_tiles, whole, (uint4 *)rec, H, mark)
    switch (variant) {
    case 0: DMS_LAUNCH(64); break;
    case 1: DMS_LAUNCH(32); break;
    default: DMS_LAUNCH(16); break;
    }
#undef DMS_LAUNCH
    queue_finish(H, rec, mark, s);
    return launch_status();
}

}  // namespace dms

extern "C" size_t dms_gradient_workspace_size(const int64_t dims[3], const int64_t lo[3],
                                              const int64_t hi[3])
{
    using namespace dms;
    if (!box_valid(dims, lo, hi) || !grid_size_values_ok(dims)) return 0;
    return gradient_workspace_size((hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2]));
}

extern "C" int dms_discrete_gradient(const int32_t *order, const int64_t dims[3], const int64_t lo[3],
                                     const int64_t hi[3], uint32_t *rec, uint32_t *critical_mask,
                                     void *workspace, size_t workspace_bytes, void *stream)
{
    using namespace dms;
    if (!box_valid(dims, lo, hi)) return DMS_E_ARG;
    if (!grid_size_ok(dims)) return DMS_E_SIZE;
    const int64_t w0 = hi[0] - lo[0], w1 = hi[1] - lo[1], w2 = hi[2] - lo[2];
    if (w0 == 0 || w1 == 0 || w2 == 0) return DMS_OK;
    if (!order || !rec) return DMS_E_ARG;
    if (workspace && workspace_bytes < gradient_workspace_size(w0 * w1 * w2)) return DMS_E_WORKSPACE;
    if (const int st = tables_ready()) return st;
    return launch_gradient_keys<RankKeys>(order, dims, lo, hi, rec, critical_mask, (char *)workspace, nullptr,
                                          (hipStream_t)stream);
}

extern "C" int dms_discrete_gradient_values(const void *values, int dtype, const int64_t dims[3],
                                            const int64_t lo[3], const int64_t hi[3], uint32_t *rec,
                                            uint32_t *critical_mask, void *workspace, size_t workspace_bytes,
                                            uint32_t *dev_flags, void *stream)
{
    using namespace dms;
    if (dtype != DMS_F32 && dtype != DMS_F64) return DMS_E_ARG;
    if (!box_valid(dims, lo, hi)) return DMS_E_ARG;
    if (!grid_size_values_ok(dims)) return DMS_E_SIZE;
    const int64_t w0 = hi[0] - lo[0], w1 = hi[1] - lo[1], w2 = hi[2] - lo[2];
    if (w0 == 0 || w1 == 0 || w2 == 0) return DMS_OK;
    if (!values || !rec || !dev_flags) return DMS_E_ARG;
    if (workspace && workspace_bytes < gradient_workspace_size(w0 * w1 * w2)) return DMS_E_WORKSPACE;
    if (const int st = tables_ready()) return st;
    if (dtype == DMS_F32)
        return launch_gradient_keys<F32Keys>(values, dims, lo, hi, rec, critical_mask, (char *)workspace,
                                             dev_flags,
                                             (hipStream_t)stream);
    return launch_gradient_keys<F64Keys>(values, dims, lo, hi, rec, critical_mask, (char *)workspace,
                                         dev_flags,
                                         (hipStream_t)stream);
}

extern "C" int dms_init(void *stream)
{
    if (const int st = dms::init_tables((hipStream_t)stream)) return st;
    return dms::init_critical_scratch();
}
