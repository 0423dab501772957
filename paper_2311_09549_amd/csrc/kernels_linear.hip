// LINEAR schedule: the perfectly nested default loop nest of an expression (Section 3, the nest a
// tensor compiler emits before any split), run as it stands: every stored entry is multiplied
// with one element of every factor for every combination of the dense output indices, nothing is
// factored out.  It is the baseline the fused and fissioned nests are compared with
// (nnz * L * M multiply-adds for the order-3 chain instead of M * (nnz + F * L), Section 1), and what
// SC_SCHED_AUTO falls back to for ranks without a factored kernel.  One workgroup per tile of
// nonzeros; the partial sum of an output row is kept in registers while the walk stays inside one
// slice.  The fp32 chain of order 3 runs as slice products (kernels_slice.hip) up to rank 128: every stored entry is a child of
// its own there.  linear_tiled_kernel takes the other expressions of order 3 and 4 at ranks that are multiples of 4;
// linear_kernel, one thread per dense output element, the other ranks and the SDDMM.
//
//   order 3 chain   A(i,l,m)   += B(i,j,k)   * C(j,l) * D(k,m)
//   MTTKRP          A(i,r)     += B(i,j,k)   * C(j,r) * D(k,r)
//   order 4 chain   A(i,l,m,n) += B(i,j,k,p) * C(j,l) * D(k,m) * E(p,n)
//   SDDMM -> SpMM   A(i,l)     += S(i,j) * X(i,k) * Y(j,k) * Z(j,l)      (loops k and l both inside)
#include "device_common.h"

#include <type_traits>

namespace sck {

namespace {

constexpr int LIN_TN = 1024;   // nonzeros per tile at most (sizes the LDS arrays)

struct LinArgs {
    const int32_t *pos[4];
    const int32_t *crd[4];
    const void *vals;
    const void *F[3];
    int64_t ld[3];
    int32_t cols[3];
    void *A;
    int32_t order, kind, row_elems;
};

// Last node x in [lo, lo + n) with pos[x] <= z: the parent of child z among the tile's nodes.
__device__ __forceinline__ int32_t parent_in(const int32_t *pos, int32_t lo, int32_t n, int32_t z)
{
    int32_t a = lo, b = lo + n - 1;
    while (a < b) {
        const int32_t mid = (a + b + 1) >> 1;
        if (pos[mid] <= z) a = mid; else b = mid - 1;
    }
    return a;
}

template <typename T>
__global__ void __launch_bounds__(NT) linear_kernel(LinArgs a, const TileRec *__restrict__ tiles)
{
    __shared__ int32_t c0_s[LIN_TN], c1_s[LIN_TN], c2_s[LIN_TN], c3_s[LIN_TN];
    __shared__ T v_s[LIN_TN];
    const TileRec t = tiles[blockIdx.x];
    const int tid = threadIdx.x;
    const int nchild = t.n1 - t.n0;
    const int d = a.order;
    const T *vals = static_cast<const T *>(a.vals);

    // coordinates of every nonzero of the tile: the leaf's own, then its ancestors' (found among the
    // tile's nodes of each level)
    for (int c = tid; c < nchild; c += NT) {
        const int32_t z = t.n0 + c;
        int32_t co[4] = {0, 0, 0, 0};
        co[d - 1] = a.crd[d - 1][z];
        const int32_t xa = parent_in(a.pos[d - 1], t.a0, t.na, z);
        co[d - 2] = a.crd[d - 2][xa];
        if (d >= 3) {
            const int32_t xb = parent_in(a.pos[d - 2], t.b0, t.nb, xa);
            co[d - 3] = a.crd[d - 3][xb];
            if (d == 4) {
                const int32_t xc = parent_in(a.pos[1], t.c0, t.nc, xb);
                co[0] = a.crd[0][xc];
            }
        }
        c0_s[c] = co[0]; c1_s[c] = co[1]; c2_s[c] = co[2]; c3_s[c] = co[3];
        v_s[c] = vals[z];
    }
    __syncthreads();

    const int E = a.row_elems;
    // E >= NT: a thread owns elements tid, tid + NT, ... and walks all nonzeros for each;
    // E <  NT: NT / E sets of E threads share the nonzeros (set s takes nonzeros s, s + sets, ...)
    const int sets = E >= NT ? 1 : NT / E;
    const int s = E >= NT ? 0 : tid / E;
    if (s >= sets) return;
    const T *F0 = static_cast<const T *>(a.F[0]), *F1 = static_cast<const T *>(a.F[1]), *F2 = static_cast<const T *>(a.F[2]);
    T *A = static_cast<T *>(a.A);
    for (int e = E >= NT ? tid : tid % E; e < E; e += (E >= NT ? NT : E)) {
        T acc = T(0);
        int32_t cur = -1;
        for (int c = s; c < nchild; c += sets) {
            const int32_t i = c0_s[c];
            if (i != cur) {
                if (cur >= 0) atomic_add(A + (int64_t)cur * E + e, acc);
                acc = T(0);
                cur = i;
            }
            const T v = v_s[c];
            switch (a.kind) {
            case K_TTMC3: {
                const int l = e / a.cols[1], m = e % a.cols[1];
                acc += v * F0[(int64_t)c1_s[c] * a.ld[0] + l] * F1[(int64_t)c2_s[c] * a.ld[1] + m];
                break;
            }
            case K_MTTKRP3:
                acc += v * F0[(int64_t)c1_s[c] * a.ld[0] + e] * F1[(int64_t)c2_s[c] * a.ld[1] + e];
                break;
            case K_TTMC4: {
                const int mn = a.cols[1] * a.cols[2];
                const int l = e / mn, m = (e / a.cols[2]) % a.cols[1], n = e % a.cols[2];
                acc += v * F0[(int64_t)c1_s[c] * a.ld[0] + l] * F1[(int64_t)c2_s[c] * a.ld[1] + m] * F2[(int64_t)c3_s[c] * a.ld[2] + n];
                break;
            }
            default: {   // K_SDDMM_SPMM: X(i,k) Y(j,k) Z(j,l), the k loop inside the l loop
                const T *x = F0 + (int64_t)i * a.ld[0], *y = F1 + (int64_t)c1_s[c] * a.ld[1];
                const T zl = F2[(int64_t)c1_s[c] * a.ld[2] + e];
                for (int k = 0; k < a.cols[0]; ++k) acc += v * x[k] * y[k] * zl;
                break;
            }
            }
        }
        if (cur >= 0) atomic_add(A + (int64_t)cur * E + e, acc);
    }
}

struct alignas(16) LinRec { uint32_t o[3]; int32_t i; };   // byte offsets of the factor rows, output row

constexpr int LIN_PADDED = LIN_TN + LIN_TN / 16;
// LDS bytes of a workgroup of linear_tiled_kernel with blocks of BX rows: records, values, a parked block and a word per thread.
// (As one struct in LDS the arrays cost the fp32 MTTKRP six registers and with them a sixth wavefront per SIMD: 306 -> 327 us on
// 20 M nonzeros at rank 32.)
template <typename T, int BX>
constexpr size_t lin_tiled_lds_bytes()
{
    return (size_t)LIN_PADDED * (sizeof(LinRec) + sizeof(T)) + (size_t)NT * (4 * BX * sizeof(T) + 4);
}

constexpr int lin_block_rows(int kind) { return kind == K_MTTKRP3 ? 1 : 4; }

// Ranks that are multiples of 4: a lane owns a 4 x 4 block of the output row (4 elements of the MTTKRP's), a lane group
// of GS lanes (the smallest power of two that covers the blocks of a row, at most a wavefront: longer rows are
// walked once per 64 blocks) walks a contiguous chunk of the tile's nonzeros.  What bounds the nest is instructions and
// gathers per nonzero, not its multiply-adds: one element per thread cost four wavefronts two 4-byte gathers and their 64-bit
// addresses per nonzero at 12 x 20 (405 us on 1.5 M nonzeros); with blocks two 16-byte gathers serve four nonzeros and 16
// multiply-adds per lane (75 us).  The pieces of a slice cut by chunk boundaries are parked in LDS and added by the
// lane group in which the slice ends; one update per tile and slice, atomic only where another tile holds part of the
// slice: one atomic update per chunk and slice made a skewed tensor's heavy slices queue on their rows (587 us).
// NARROW, rows of at most 8 blocks: up to 256 lane groups, so the pieces of a heavy slice make a long chain.  They are added
// up inside the wavefronts first: 200 slices of 1,500 nonzeros at 4 x 4 took 61 us, 34 us with one element per
// thread, 16 us so; the MTTKRP at rank 4 41, 29 and 14 us.  Wider rows gain less than the steps cost (12 x 20: 37.2 -> 38.0 us).
template <typename T, int KIND, bool NARROW>
__global__ void __launch_bounds__(NT) linear_tiled_kernel(LinArgs a, const TileRec *__restrict__ tiles)
{
    constexpr int U = 4;                                 // nonzeros per step
    constexpr int BX = lin_block_rows(KIND);
    constexpr int D = KIND == K_TTMC4 ? 4 : 3;
    struct alignas(16) V4 { T v[4]; };   // the rows of the factors are 16-byte aligned
    using Rec = LinRec;
    // records of chunks that start a multiple of 16 apart spread over the banks
    auto at = [](int c) { return c + (c >> 4); };
    __shared__ Rec rec_s[LIN_PADDED];
    __shared__ T v_s[LIN_PADDED];
    __shared__ T park_s[4 * BX][NT];    // the open sum of every chunk ...
    __shared__ int32_t began_s[NT];     // ... bit 0: the slice began in a chunk that this sum holds, bit 1: summed over the wavefront
    static_assert(sizeof(rec_s) + sizeof(v_s) + sizeof(park_s) + sizeof(began_s) == lin_tiled_lds_bytes<T, BX>(), "reported LDS");
    static_assert(lin_tiled_lds_bytes<T, BX>() <= 64 * 1024, "LDS of a workgroup");
    const TileRec t = tiles[blockIdx.x];
    const int tid = threadIdx.x;
    const int nchild = t.n1 - t.n0;
    const T *vals = static_cast<const T *>(a.vals);
    for (int c = tid; c < nchild; c += NT) {
        const int32_t z = t.n0 + c;
        int32_t x = z;
        Rec r;
        r.o[2] = 0;
        r.o[D - 2] = (uint32_t)a.crd[D - 1][z] * (uint32_t)(a.ld[D - 2] * sizeof(T));
        x = parent_in(a.pos[D - 1], t.a0, t.na, x);
        r.o[D - 3] = (uint32_t)a.crd[D - 2][x] * (uint32_t)(a.ld[D - 3] * sizeof(T));
        x = parent_in(a.pos[D - 2], t.b0, t.nb, x);
        if (D == 4) {
            r.o[0] = (uint32_t)a.crd[1][x] * (uint32_t)(a.ld[0] * sizeof(T));
            x = parent_in(a.pos[1], t.c0, t.nc, x);
        }
        r.i = a.crd[0][x];
        rec_s[at(c)] = r;
        v_s[at(c)] = vals[z];
    }
    __syncthreads();

    const int E = a.row_elems, nblk = E / (4 * BX);
    int gs_log = 0;
    while ((1 << gs_log) < nblk && gs_log < 6) ++gs_log;
    const int G = NT >> gs_log, g = tid >> gs_log, li = tid & ((1 << gs_log) - 1);
    const int q = (nchild + G - 1) / G, c0 = min(g * q, nchild), c1 = min(c0 + q, nchild);
    const bool some = c0 < c1;
    // the chunk's first slice began in an earlier chunk / its last slice goes on in the next one
    const bool cont = some && c0 > 0 && rec_s[at(c0 - 1)].i == rec_s[at(c0)].i;
    const bool open = some && c1 < nchild && rec_s[at(c1)].i == rec_s[at(c1 - 1)].i;
    // slices shared with the neighbouring tiles
    const int32_t i_in = (t.flags & (D == 4 ? 16 : 4)) ? rec_s[at(0)].i : -1, i_out = (t.flags & (D == 4 ? 32 : 8)) ? rec_s[at(nchild - 1)].i : -1;
    T *A = static_cast<T *>(a.A);
    const char *F0 = static_cast<const char *>(a.F[0]), *F1 = static_cast<const char *>(a.F[1]), *F2 = static_cast<const char *>(a.F[2]);
    for (int pass = 0; pass < nblk; pass += 1 << gs_log) {
        const int blk = min(pass + li, nblk - 1);
        const bool mine = some && pass + li < nblk;
        // block -> byte offsets of its pieces in the factor rows, first element and row distance in the output row
        uint32_t p0 = 0, p1 = 0, p2 = 0;
        int e0, dist = 0;
        if (KIND == K_MTTKRP3) {
            e0 = 4 * blk;
            p0 = p1 = (uint32_t)(e0 * sizeof(T));
        } else if (KIND == K_TTMC3) {
            const int n4 = a.cols[1] / 4, x = blk / n4, y = blk % n4;
            p0 = (uint32_t)(4 * x * sizeof(T));
            p1 = (uint32_t)(4 * y * sizeof(T));
            dist = a.cols[1];
            e0 = 4 * x * dist + 4 * y;
        } else {
            const int m4 = a.cols[1] / 4, n4 = a.cols[2] / 4, l = blk / (m4 * n4), x = blk / n4 % m4, y = blk % n4;
            p0 = (uint32_t)(l * sizeof(T));
            p1 = (uint32_t)(4 * x * sizeof(T));
            p2 = (uint32_t)(4 * y * sizeof(T));
            dist = a.cols[2];
            e0 = (l * a.cols[1] + 4 * x) * dist + 4 * y;
        }
        T acc[BX][4];
#pragma unroll
        for (int x = 0; x < BX; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) acc[x][y] = T(0);
        bool first = cont;       // still in the slice that began in an earlier chunk
        int32_t cur = -1, head_i = -1;
        T head[BX][4];
#pragma unroll
        for (int x = 0; x < BX; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) head[x][y] = T(0);
        auto emit = [&](int32_t i, const T (&o)[BX][4]) {
            T *dst = A + (int64_t)i * E + e0;
#pragma unroll
            for (int x = 0; x < BX; ++x) {
                V4 w;
#pragma unroll
                for (int y = 0; y < 4; ++y) w.v[y] = o[x][y];
                if (i != i_in && i != i_out) {
                    *reinterpret_cast<V4 *>(dst + x * dist) = w;
                } else {
#pragma unroll
                    for (int y = 0; y < 4; ++y) atomic_add(dst + x * dist + y, w.v[y]);
                }
            }
        };
        auto end_slice = [&]() {
            if (first) {
#pragma unroll
                for (int x = 0; x < BX; ++x)
#pragma unroll
                    for (int y = 0; y < 4; ++y) head[x][y] = acc[x][y];
                head_i = cur;
            } else {
                emit(cur, acc);
            }
            first = false;
#pragma unroll
            for (int x = 0; x < BX; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) acc[x][y] = T(0);
        };
        if (mine) {
            cur = rec_s[at(c0)].i;
            for (int c = c0; c < c1; c += U) {
                Rec r[U];
                T v[U], s[U];
                V4 x[U], y[U];
    #pragma unroll
                for (int u = 0; u < U; ++u) {   // steps past the chunk repeat its last nonzero and are not added
                    r[u] = rec_s[at(min(c + u, c1 - 1))];
                    v[u] = v_s[at(min(c + u, c1 - 1))];
                }
    #pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (KIND == K_TTMC4) {
                        s[u] = *reinterpret_cast<const T *>(F0 + (r[u].o[0] + p0));
                        x[u] = *reinterpret_cast<const V4 *>(F1 + (r[u].o[1] + p1));
                        y[u] = *reinterpret_cast<const V4 *>(F2 + (r[u].o[2] + p2));
                    } else {
                        x[u] = *reinterpret_cast<const V4 *>(F0 + (r[u].o[0] + p0));
                        y[u] = *reinterpret_cast<const V4 *>(F1 + (r[u].o[1] + p1));
                    }
                }
    #pragma unroll
                for (int u = 0; u < U; ++u)
                    if (c + u < c1) {
                        if (r[u].i != cur) {
                            end_slice();
                            cur = r[u].i;
                        }
                        const T vs = KIND == K_TTMC4 ? v[u] * s[u] : v[u];
                        if (KIND == K_MTTKRP3) {
    #pragma unroll
                            for (int k = 0; k < 4; ++k) acc[0][k] += vs * x[u].v[k] * y[u].v[k];
                        } else {
    #pragma unroll
                            for (int k = 0; k < BX; ++k) {
                                const T vx = vs * x[u].v[k];
    #pragma unroll
                                for (int n = 0; n < 4; ++n) acc[k][n] += vx * y[u].v[n];
                            }
                        }
                    }
            }
            if (!open) end_slice();
        }
        // ---- slices cut by chunk boundaries ----
        if (pass) __syncthreads();   // the previous pass's pieces have been read
        int began = !first;
        if constexpr (NARROW) {
            // four chunks in a row (eight of one or two lanes) that lie inside one slice: the wavefront's open sums are added up by doubling
            // steps, each from the chunk where its slice began or, if that is in an earlier wavefront, from the wavefront's first chunk
            const unsigned long long inside = __ballot(some && first && open);
            const int gs = 1 << gs_log;
            unsigned long long row = inside & (inside >> gs);
            row &= row >> 2 * gs;
            if (gs <= 2) row &= row >> 4 * gs;
            if (row) {
#pragma unroll
                for (int x = 0; x < BX; ++x)
#pragma unroll
                    for (int y = 0; y < 4; ++y) acc[x][y] = mine && open ? acc[x][y] : T(0);
                const int lane = tid % 64;
                for (int d = gs; d < 64; d <<= 1) {
                    const int before = __shfl_up(began, d);
                    const bool add = lane >= d && !began;
#pragma unroll
                    for (int x = 0; x < BX; ++x)
#pragma unroll
                        for (int y = 0; y < 4; ++y) {
                            const T o = __shfl_up(acc[x][y], d);
                            acc[x][y] += add ? o : T(0);
                        }
                    began |= lane >= d && before;
                }
                began |= 2;
            }
        }
        if (mine && open) {
#pragma unroll
            for (int x = 0; x < BX; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) park_s[4 * x + y][tid] = acc[x][y];
        }
        if (li == 0) began_s[g] = began;
        __syncthreads();
        if (head_i >= 0) {
            for (int h = g - 1; h >= 0; --h) {
#pragma unroll
                for (int x = 0; x < BX; ++x)
#pragma unroll
                    for (int y = 0; y < 4; ++y) head[x][y] += park_s[4 * x + y][(h << gs_log) + li];
                const int b = began_s[h];
                if (b & 1) break;                                           // the slice began in chunk h ...
                if (NARROW && b) h = ((h << gs_log) & ~63) >> gs_log;       // ... or the sum reaches back to the wavefront's first chunk
            }
            emit(head_i, head);
        }
    }
}

// Chains whose last two ranks, and MTTKRPs whose rank, are multiples of 4 run linear_tiled_kernel: 405 -> 75 us at 12 x 20.
bool linear_is_tiled(const sc_plan *p)
{
    switch (p->kind) {
    case K_TTMC3:
    case K_MTTKRP3: return p->fcols[0] % 4 == 0 && p->fcols[1] % 4 == 0;
    case K_TTMC4: return p->fcols[1] % 4 == 0 && p->fcols[2] % 4 == 0;
    default: return false;
    }
}

template <typename T>
void launch_linear_nest(const sc_plan *p, const LinArgs &a, int ntiles, hipStream_t stream)
{
    const int nblk = a.row_elems / (4 * lin_block_rows(p->kind));
    auto tiled = [&](auto kind) {
        constexpr int KIND = decltype(kind)::value;
        if (nblk <= 8) linear_tiled_kernel<T, KIND, true><<<ntiles, NT, 0, stream>>>(a, p->d_tiles);
        else linear_tiled_kernel<T, KIND, false><<<ntiles, NT, 0, stream>>>(a, p->d_tiles);
    };
    const bool blocks = linear_is_tiled(p);
    if (blocks && p->kind == K_TTMC3) tiled(std::integral_constant<int, K_TTMC3>{});
    else if (blocks && p->kind == K_MTTKRP3) tiled(std::integral_constant<int, K_MTTKRP3>{});
    else if (blocks && p->kind == K_TTMC4) tiled(std::integral_constant<int, K_TTMC4>{});
    else linear_kernel<T><<<ntiles, NT, 0, stream>>>(a, p->d_tiles);
}

}  // namespace

size_t linear_lds_bytes(const sc_plan *p)
{
    if (p->caps.tn > LIN_TN) return SIZE_MAX;
    const bool f64 = p->dtype == SC_F64;
    if (!linear_is_tiled(p)) return (size_t)LIN_TN * (16 + (f64 ? 8 : 4));   // four coordinates and the value
    if (lin_block_rows(p->kind) == 1) return f64 ? lin_tiled_lds_bytes<double, 1>() : lin_tiled_lds_bytes<float, 1>();
    return f64 ? lin_tiled_lds_bytes<double, 4>() : lin_tiled_lds_bytes<float, 4>();
}

sc_status launch_linear(const sc_plan *p, const sc_csf_view *sp, const sc_dense_view *fac, void *out, hipStream_t stream)
{
    Launcher ln{p, stream};
    if (p->dtype == SC_F64)
        launch_output_zero<double>(ln, p, static_cast<double *>(out));
    else
        launch_output_zero<float>(ln, p, static_cast<float *>(out));
    const int ntiles = (int)p->tiles.size();
    if (ntiles == 0) return ln.status;
    if (p->caps.tn > LIN_TN) return SC_ERR_SCHED_UNSUPPORTED;
    if (plan_slice_source(p, nullptr) != SLICE_NONE) return launch_slice(p, ln, sp, fac[0], &fac[1], nullptr, fac[1].cols, out, "linear_nest");
    LinArgs a = {};
    for (int m = 0; m < 4; ++m) {
        a.pos[m] = sp->pos[m];
        a.crd[m] = sp->crd[m];
    }
    a.vals = sp->vals;
    for (int s = 0; s < p->nfactors; ++s) {
        a.F[s] = fac[s].data;
        a.ld[s] = fac[s].ld;
        a.cols[s] = (int32_t)fac[s].cols;
    }
    a.A = out;
    a.order = p->order;
    a.kind = (int32_t)p->kind;
    a.row_elems = (int32_t)p->out_row_elems;
    ln.begin("linear_nest");
    if (p->dtype == SC_F64)
        launch_linear_nest<double>(p, a, ntiles, stream);
    else
        launch_linear_nest<float>(p, a, ntiles, stream);
    ln.end();
    return ln.status;
}

}  // namespace sck
