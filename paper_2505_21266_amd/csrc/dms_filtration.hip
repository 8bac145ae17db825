// dms_filtration.hip -- critical cells of one dimension in the filtration
// order of Section 2.1: a cell's key is the list of its vertex orders sorted
// decreasingly, and keys of one dimension compare lexicographically.
//
// Two cells compare by their highest vertices' orders unless they share that
// vertex w; then their other vertices are neighbours of w, and their orders
// compare like their ranks among w's (at most 14) neighbours.  So the key is
// the order of w (32 bits) above the ranks of the other vertices, decreasing,
// 4 bits each: at most 44 bits, ranked by one radix sort of 4 to 6 passes
// (two 64-bit words of plain orders took 8 passes for vertices and edges and
// 16 for triangles and tets).
#include "dms_common.hpp"
#include "dms_internal.hpp"
#include "dms_tables.hpp"

namespace dms {
namespace {

constexpr int kThreads = 256;

// The star geometry a cell code refers to (kernel argument).
struct Geom {
    int8_t nb[14][3];  // (dx, dy, dz) of neighbour e
    uint8_t tri[36][2];
    uint8_t tet[24][3];
};

Geom make_geom()
{
    Geom g{};
    const Tables &T = kTables;
    for (int e = 0; e < 14; ++e)
        for (int c = 0; c < 3; ++c) g.nb[e][c] = (int8_t)T.nb[e][c];
    for (int t = 0; t < 36; ++t)
        for (int c = 0; c < 2; ++c) g.tri[t][c] = (uint8_t)T.tri[t][c];
    for (int q = 0; q < 24; ++q)
        for (int c = 0; c < 3; ++c) g.tet[q][c] = (uint8_t)T.tet[q][c];
    return g;
}

// Bits of a dimension's keys.
constexpr int key_bits(int dim) { return 32 + 4 * dim; }

// Keys of the cells: code = (maxv << 8) | local index (0 for a vertex,
// neighbour e for an edge, star triangle t, star tet q).  A code naming no
// cell of the grid gets the largest key and raises DMS_FLAG_BADCODE.
__global__ __launch_bounds__(kThreads) void k_cell_keys(const int64_t *__restrict__ codes, int64_t count,
                                                        int dim, const int32_t *__restrict__ order,
                                                        int64_t nx, int64_t ny, int64_t nz, Geom g,
                                                        uint64_t *__restrict__ key, uint32_t *flags)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= count) return;
    const int64_t code = codes[i];
    const int64_t v = code >> 8;
    const int loc = (int)(code & 255);
    const int64_t n = nx * ny * nz;
    int oth[3] = {0, 0, 0};
    bool bad = v < 0 || v >= n;
    if (dim == 0) {
        bad = bad || loc != 0;
    } else if (dim == 1) {
        bad = bad || loc >= 14;
        oth[0] = loc < 14 ? loc : 0;
    } else if (dim == 2) {
        bad = bad || loc >= 36;
        const int t = loc < 36 ? loc : 0;
        oth[0] = g.tri[t][0];
        oth[1] = g.tri[t][1];
    } else {
        bad = bad || loc >= 24;
        const int q = loc < 24 ? loc : 0;
        oth[0] = g.tet[q][0];
        oth[1] = g.tet[q][1];
        oth[2] = g.tet[q][2];
    }
    uint32_t o[4] = {0u, 0u, 0u, 0u};
    uint64_t k = 0;
    if (!bad) {
        const int64_t x = v % nx, y = (v / nx) % ny, z = v / (nx * ny);
        int64_t tx = x, ty = y, tz = z;  // the highest vertex
        o[0] = (uint32_t)order[v];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (c >= dim) continue;
            const int e = oth[c];
            const int64_t a = x + g.nb[e][0], b = y + g.nb[e][1], d = z + g.nb[e][2];
            if (a < 0 || b < 0 || d < 0 || a >= nx || b >= ny || d >= nz) {
                bad = true;
                continue;
            }
            o[c + 1] = (uint32_t)order[a + nx * (b + ny * d)];
            if (o[c + 1] > o[0]) {  // (not so for codes as the extraction writes them)
                const uint32_t s = o[0];
                o[0] = o[c + 1];
                o[c + 1] = s;
                tx = a;
                ty = b;
                tz = d;
            }
        }
        // ranks of the other vertices among the highest one's neighbours
        uint32_t r[3] = {0u, 0u, 0u};
        if (!bad && dim > 0) {
#pragma unroll
            for (int e = 0; e < 14; ++e) {
                const int64_t a = tx + g.nb[e][0], b = ty + g.nb[e][1], d = tz + g.nb[e][2];
                if (a < 0 || b < 0 || d < 0 || a >= nx || b >= ny || d >= nz) continue;
                const uint32_t w = (uint32_t)order[a + nx * (b + ny * d)];
#pragma unroll
                for (int c = 0; c < 3; ++c) r[c] += w < o[c + 1] ? 1u : 0u;
            }
        }
        // decreasing; the absent ones (0) stay last
        uint32_t hi = r[0] > r[1] ? r[0] : r[1], mid = r[0] > r[1] ? r[1] : r[0], low = r[2];
        if (dim == 3) {
            if (low > mid) { const uint32_t s = mid; mid = low; low = s; }
            if (mid > hi) { const uint32_t s = hi; hi = mid; mid = s; }
        }
        const uint32_t local = dim == 0 ? 0u : dim == 1 ? hi : dim == 2 ? hi << 4 | mid : hi << 8 | mid << 4 | low;
        k = (uint64_t)o[0] << (4 * dim) | local;
    }
    if (bad) {
        atomicOr(flags, (uint32_t)DMS_FLAG_BADCODE);
        k = (1ull << key_bits(dim)) - 1ull;
    }
    key[i] = k;
}

// out_codes[rank[i]] = in_codes[i].
__global__ __launch_bounds__(kThreads) void k_cell_place(const int32_t *__restrict__ rank, int64_t count,
                                                         const int64_t *__restrict__ in_codes,
                                                         int64_t *__restrict__ out_codes)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= count) return;
    const int32_t r = rank[i];
    if (r >= 0 && r < count) out_codes[r] = in_codes[i];
}

struct RankLayout {
    size_t key, rws, total;
};

RankLayout rank_layout(int64_t count)
{
    const size_t c = (size_t)(count > 0 ? count : 1);
    RankLayout L{};
    size_t off = 0;
    L.key = off; off += align_up(c * 8, 256);
    L.rws = off; off += rank_u64_workspace_size(count);
    L.total = off;
    return L;
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

size_t cell_rank_workspace_size(int64_t count) { return rank_layout(count).total; }

int launch_cell_ranks(const int64_t *codes, int64_t count, int dim, const int32_t *order, const int64_t *dims,
                      int32_t *rank, char *ws, uint32_t *flags, hipStream_t s)
{
    if (count == 0) return DMS_OK;
    const RankLayout L = rank_layout(count);
    uint64_t *key = (uint64_t *)(ws + L.key);
    hipLaunchKernelGGL(k_cell_keys, dim3(blocks_for(count)), dim3(kThreads), 0, s, codes, count, dim, order, dims[0],
                       dims[1], dims[2], make_geom(), key, flags);
    return launch_rank_u64(key, count, key_bits(dim), rank, ws + L.rws, flags, s);
}

}  // namespace dms

namespace {
size_t sort_rank_offset(int64_t count)
{
    return dms::align_up((size_t)(count > 0 ? count : 1) * 4, 256);
}
}  // namespace

extern "C" size_t dms_critical_sort_workspace_size(int64_t count)
{
    if (count < 0) return 0;
    return sort_rank_offset(count) + dms::cell_rank_workspace_size(count);
}

extern "C" int dms_critical_sort(const int64_t *codes, int64_t count, int dim, const int32_t *order,
                                 const int64_t dims[3], int64_t *sorted, void *workspace,
                                 size_t workspace_bytes, uint32_t *dev_flags, void *stream)
{
    using namespace dms;
    if (!dims || dims[0] < 1 || dims[1] < 1 || dims[2] < 1 || count < 0 || dim < 0 || dim > 3)
        return DMS_E_ARG;
    if (!grid_size_ok(dims)) return DMS_E_SIZE;
    if (count > 2147483647LL) return DMS_E_SIZE;
    if (count == 0) return DMS_OK;
    if (!codes || !order || !sorted || !dev_flags || sorted == codes) return DMS_E_ARG;
    if (!workspace || workspace_bytes < dms_critical_sort_workspace_size(count)) return DMS_E_WORKSPACE;
    if (const int dc = device_check()) return dc;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)workspace;
    int32_t *rank = (int32_t *)ws;
    const int st = launch_cell_ranks(codes, count, dim, order, dims, rank, ws + sort_rank_offset(count),
                                     dev_flags, s);
    if (st) return st;
    hipLaunchKernelGGL(k_cell_place, dim3(blocks_for(count)), dim3(kThreads), 0, s, rank, count, codes,
                       sorted);
    return launch_status();
}
