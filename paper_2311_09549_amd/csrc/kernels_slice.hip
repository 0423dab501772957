// Slice products on matrix cores, fp32: the last contraction of a TTM chain,
//     A(i,:,:) = sum over the children f of slice i of  C(j_f,:)^T (x) T(f,:)          (L x W per slice)
// with the rows of T either formed on the way from the leaves of the tensor (FUSED, and the unfactored nest: Table 2,
// kernel 6 <SpTTM, TTM>; also the sparse part of kernel 5) or read from the workspace (the last kernel of the FISSIONED
// schedules of order 3 and 4).
//
// Four children form a step group, the K = 4 of v_mfma_f32_16x16x4_f32: lanes 16 kk .. 16 kk + 15 hold the row of child kk.
// Which l and m a tile's rows and columns stand for is free, so a lane reads MT adjacent values of a row of T (or of D) and LT
// adjacent values of a row of C straight into operand registers: no row of T passes through LDS.  A wavefront owns a run of
// steps and all (or a half, quarter) of the L x W output of the slice it is in; it shares nothing with its neighbours, so
// there is no barrier, and wavefronts in different phases keep the gathers and the matrix cores busy together.
//
//   SRC_LEAVES  the plan lists for every step the leaf that each of the four fibers of the group contributes: its last coordinate
//               and the place of its value among the values of the chunk of steps (64 at most), which are contiguous.  Fibers are
//               cut into pieces of at most kSlicePiece leaves and grouped by length inside a chunk's part of a slice.
//               t(f,:) += B * D(k,:) stays in MT registers until the group's last step.
//   SRC_ROWS    a step is four consecutive children; their rows of T are 4 W adjacent floats in memory.
//
// A run ends anywhere in a slice (runs have equal work): a slice inside one run is stored once, a slice cut by a run's end
// is added to the zeroed row atomically, after the runs of a workgroup that lie inside one slice have been added up in LDS.  A chunk is staged
// in a region of LDS of the wavefront's own ({row offset, value} per leaf, offset of C(j,:) per child), read a chunk ahead; the loop
// then takes U steps per batch, whose gathers are all issued before the first is used.
#include "slice_common.h"

#include <type_traits>

namespace sck {

namespace {

constexpr int SRC_LEAVES = 0, SRC_ROWS = 1;

// Whether the rows of the output are stored with the non-temporal hint.  Written through the L2s they evict the rows of C and D that the
// gathers hit there, which costs most where a slice gathers much for what it stores, and an output beyond the memory-side cache (256 MB)
// evicts the rows that the launch before has zeroed there; but stores with the hint are slow in pieces of less than a cache line, and they
// do not stay in that cache for whoever reads or writes the output next.  Repeated calls on uniform tensors from leaves, us without the hint and
// with it, at 64 x 64, 16 x 16 and 64 x 16:
//     entries per slice             1 or 2                    3                         8                         14 to 18
//     150 to 180 MB                 36,41  35,39  27,31       40,47  38,43  33,48       45,47  41,48  40,51       51,50  61,54  44,44
//     300 MB, a third stored        64,61  61,60  55,65
//             all stored                                      69,71  69,69  69,98       70,74  86,77  71,99       79,80  112,81  87,87
//     400 MB, a third stored        92,70  97,74  92,85
//             all stored                                      92,92  93,92  88,135      98,95  116,96  102,128    128,122  174,105  139,113
//     400 MB, more than three quarters of the rows empty, so that the whole output is zeroed first, five entries: 110,121  97,109
// From rows of T, which are read once and evict as well: 300 MB, 3 per slice, 16 x 16 125 and 118, 64 x 16 101 and 93, 128 x 16 85 and 95; 8 per
// slice, 128 x 16 126 and 115; 16 x 16 at 180 MB, 14 per slice, 154 and 130.
bool stores_past_caches(int64_t bytes, bool all_zeroed, int64_t stored, double per_slice, int64_t L, int64_t W, bool rows)
{
    constexpr int64_t MB = 1 << 20;
    const bool one_tile = L <= 16 && W <= 16;   // a slice is one piece
    if (W % 16 != 0 && !one_tile) return false;
    if (stored > 128 * MB && per_slice >= (one_tile || (rows && L <= 16) ? 12 : 16)) return true;
    if (bytes <= 256 * MB || all_zeroed) return false;
    if (rows) return L <= 64 || W > 16 || per_slice >= 8;
    if (W % 32 != 0 && !one_tile) return false;
    return bytes > 384 * MB || bytes - stored > bytes / 8 || one_tile || (L <= 16 && per_slice >= 8);
}

struct SliceArgs {
    int32_t nruns;
    const uint32_t *leaf, *at;   // SRC_LEAVES: 4 last coordinates per step, 4 places of the value in the chunk (bytes)
    const int32_t *gj;           // SRC_LEAVES: 4 per group, coordinate of the row of C
    const int32_t *first;        // SRC_ROWS: first child of every step and the child count
    const int32_t *crd1;         // output row of every slice
    const int32_t *crd2;         // SRC_ROWS: coordinate of the row of C of every child
    int32_t nslices;
    const float *vals;           // SRC_LEAVES
    const float *C, *D;          // D: SRC_LEAVES the factor of the last mode, SRC_ROWS the rows of T
    uint32_t rowC, rowD;         // bytes from row to row
    uint32_t bytesC, bytesD;     // size of C; of D (SRC_ROWS: reach of the 32-bit offsets from a run's first child)
    float *A;
    int32_t L, W;
    int32_t stream;              // the output is stored past the L2s
};

// Steps per batch and wavefronts per SIMD by the number of 16 x 16 tiles.  Repeated calls: one tile, 4 M leaves, 46.5 us with eight steps,
// 43.7 with four; eight tiles, 6 M leaves at 64 x 32, 227 us with eight steps and three wavefronts, 239 with four steps, 240 with two
// wavefronts, 410 with four, whose registers spill; sixteen: what two wavefronts have registers for.
constexpr int slice_batch(int tiles) { return tiles == 1 || tiles == 16 ? 4 : 8; }
constexpr int slice_occupancy(int tiles, bool edge) { return tiles == 16 ? 2 : (tiles == 8 ? 3 : 4) - (edge ? 1 : 0); }

// runs: nruns + 1 records, chunks: one past the last.  Arguments of their own, so that the loop reads them through the scalar cache.
// LT, MT: 16-wide tiles of l and m per wavefront; WL x WM wavefronts share a run; EDGE: L or W may be less than the tiles cover.
template <int LT, int MT, int WL, int WM, int SRC, bool EDGE>
__global__ void __launch_bounds__(NT, slice_occupancy(LT * MT, EDGE)) slice_kernel(SliceArgs a, const SliceRun *__restrict__ runs,
                                                                                      const SliceChunk *__restrict__ chunks)
{
    constexpr int WPR = WL * WM;              // wavefronts per run
    constexpr int WAVES = NT / 64;
    constexpr int RPB = WAVES / WPR;          // runs per workgroup
    constexpr int U = slice_batch(LT * MT);   // steps per batch
    constexpr bool TURNED = LT * MT == 1;     // which of l and m runs over the registers of an accumulator
    typedef float TVec __attribute__((ext_vector_type(MT)));
    typedef float CVec __attribute__((ext_vector_type(LT)));
    struct alignas(8) Rec { uint32_t off; float v; };

    struct Own {                          // a wavefront's own staging region
        alignas(16) Rec rec[256];
        uint32_t coff[256];
        float swap[256];                  // the chunk's values while it is staged; a row on its way to atomic additions
    };
    union Lds {
        Own own[WAVES];
        sl_floatx4 sum[2][RPB > 1 ? 64 * LT * MT : 1];   // after the runs: sums on their way to another wavefront
    };
    __shared__ Lds lds;
    __shared__ int state_s[WAVES];
    static_assert(sizeof(Lds) + sizeof(state_s) <= kSliceLdsBytes, "LDS the plan reports");

    const int wave = sl_uni(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int kk = lane / 16, col = lane % 16;
    const int run = (int)blockIdx.x * RPB + wave / WPR, sub = wave % WPR;
    Rec *rec_s = lds.own[wave].rec;
    uint32_t *coff_s = lds.own[wave].coff;
    float *swap_s = lds.own[wave].swap;
    const int L = EDGE ? a.L : 16 * LT * WL, W = EDGE ? a.W : 16 * MT * WM;
    const int l0 = (sub / WM) * 16 * LT, m0 = (sub % WM) * 16 * MT;
    // first of the lane's values of l and m; lanes past a row read its end again and are not stored
    const int ll = l0 + LT * col, lm = m0 + MT * col;
    // 32-bit byte offsets: one addition per gather
    const uint32_t c_lane = 4 * (EDGE ? min(ll, L - LT) : ll), d_lane = 4 * (EDGE ? min(lm, W - MT) : lm);
    const char *Db = reinterpret_cast<const char *>(a.D);

    // a wavefront past the last run has no steps
    const SliceRun r = runs[min(run, a.nruns)], r_end = runs[min(run + 1, a.nruns)];
    const int c_end = r_end.chunk0 + (r_end.step > 0 ? 1 : 0);   // one past the last chunk of which this run has steps
    SliceChunk ch = chunks[r.chunk0];
    auto below = [](uint64_t bits, int n) { return __builtin_popcountll(bits & ((1ull << n) - 1)); };   // n < 64
    const int slice0 = ch.slice0 + below(ch.send, r.step);
    int sl = slice0;
    bool open = (r.flags & 1) != 0;   // the slice began in an earlier run
    int fbase = 0;
    if (SRC == SRC_ROWS && r.chunk0 < c_end) {
        fbase = sl_uni(a.first[ch.step0 + r.step]);
        Db += (int64_t)fbase * a.rowD;
    }
    const __amdgpu_buffer_rsrc_t rowsC = sl_rows(a.C, a.bytesC), rowsD = sl_rows(Db, a.bytesD);

    // Global reads of a chunk's staging: lane n takes step n (those past the chunk repeat its last one) and the group that step belongs
    // to.  They are issued a chunk ahead and land while the one before is worked on.
    struct Stage {
        uint4 leaf;
        uint32_t at;
        int4 j;
        float v[4];
        int f0, f1, row;
    };
    auto issue = [&](const SliceChunk &k, Stage &s) {
        const int n = min(lane, k.nsteps - 1);
        s.row = a.crd1[min(k.slice0 + lane, a.nslices - 1)];   // the output rows of the slices the chunk may complete
        if (SRC == SRC_LEAVES) {
            s.leaf = reinterpret_cast<const uint4 *>(a.leaf)[k.step0 + n];
            s.at = a.at[k.step0 + n];
            const int g = __builtin_amdgcn_mbcnt_hi((uint32_t)(k.gend >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)k.gend, 0));   // groups completed before step `lane`
            s.j = reinterpret_cast<const int4 *>(a.gj)[k.group0 + min(g, k.ngroups - 1)];
#pragma unroll
            for (int q = 0; q < 4; ++q) s.v[q] = a.vals[k.leaf0 + min(64 * q + lane, k.nleaves - 1)];
        } else {
            s.f0 = a.first[k.step0 + n];
            s.f1 = a.first[k.step0 + n + 1];   // 1 to 4 children
            s.j.x = a.crd2[s.f0];
            s.j.y = a.crd2[min(s.f0 + 1, s.f1 - 1)];
            s.j.z = a.crd2[min(s.f0 + 2, s.f1 - 1)];
            s.j.w = a.crd2[min(s.f0 + 3, s.f1 - 1)];
        }
    };

    // Sums of up to SPAN steps, and sums of those.  One chain of additions over a run, hundreds of steps long in a heavy slice, was up to 2.3
    // times further from the sum in double precision than the tile by tile sums it replaces; so 64 x 64 values are
    // shared by two wavefronts, though one would hold them once (64 x 32, 6 M leaves: call of 227 us, 219 with one set of sums).
    constexpr int SPAN = 16;
    sl_floatx4 acc[MT][LT], tot[MT][LT];
    auto clear = [&](auto &v) {
        for (auto &row : v)
            for (sl_floatx4 &e : row) e = sl_floatx4{0.f, 0.f, 0.f, 0.f};
    };
    auto gather_sums = [&](sl_floatx4 (&to)[MT][LT], const sl_floatx4 (&from)[MT][LT]) {
#pragma unroll
        for (int x = 0; x < MT; ++x)
#pragma unroll
            for (int y = 0; y < LT; ++y) to[x][y] += from[x][y];
    };
    TVec t;
#pragma unroll
    for (int x = 0; x < MT; ++x) t[x] = 0.f;
    clear(acc);
    clear(tot);

    auto multiply = [&](const TVec &tv, const CVec &cv) {
#pragma unroll
        for (int x = 0; x < MT; ++x)
#pragma unroll
            for (int y = 0; y < LT; ++y)
                acc[x][y] = TURNED ? __builtin_amdgcn_mfma_f32_16x16x4f32(tv[x], cv[y], acc[x][y], 0, 0, 0)
                                   : __builtin_amdgcn_mfma_f32_16x16x4f32(cv[y], tv[x], acc[x][y], 0, 0, 0);
    };
    // acc[x][y][q] = A(l = l0 + LT (4 kk + q) + y, m = lm + x): a store instruction covers four rows l of 16 MT adjacent floats.
    // One tile: acc[0][0][q] = A(l = col, m = 4 kk + q), one store instruction for the slice (from rows of T at 16 x 16, 150,000 entries in
    // 55,000 slices: 24.5 us the other way and 21 so; at 64 x 16, 400 MB, two to four rows apart in the same layout 98 and 104).
    constexpr int STORE = 0, STREAM = 1, ADD = 2;
    auto emit = [&](int row, auto how) {
        constexpr int HOW = decltype(how)::value;
        float *A = a.A + (int64_t)row * L * W;
        if constexpr (TURNED) {
            if (HOW != ADD) {
                sl_floatx4 *dst = reinterpret_cast<sl_floatx4 *>(A + col * W + 4 * kk);
                if (HOW == STREAM) __asm__ volatile("" : "+v"(dst));   // kept apart from the plain store: merged into one, the hint is lost
                if (!EDGE || (col < L && 4 * kk < W)) {
                    if (HOW == STREAM) __builtin_nontemporal_store(acc[0][0], dst);
                    else *dst = acc[0][0];
                }
            } else {
                // adjacent lanes on adjacent floats: the four of a lane one after the other visit every cache line four times
                sl_lanes_meet();
                *reinterpret_cast<sl_floatx4 *>(swap_s + 16 * col + 4 * kk) = acc[0][0];
                sl_lanes_meet();
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int l = 4 * q + kk;
                    const float v = swap_s[64 * q + lane];
                    if (!EDGE || (l < L && col < W)) atomic_add(A + l * W + col, v);
                }
            }
            return;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)   // (y inside: adjacent rows right after each other, 64 x 8 at 140 MB 135 us the other way and 73 so)
#pragma unroll
            for (int y = 0; y < LT; ++y) {
                const int l = l0 + LT * (4 * kk + q) + y;
                TVec o;
#pragma unroll
                for (int x = 0; x < MT; ++x) o[x] = acc[x][y][q];
                if (HOW != ADD) {
                    TVec *dst = reinterpret_cast<TVec *>(A + l * W + lm);
                    if (!EDGE || (l < L && lm < W)) {
                        if (HOW == STREAM) __builtin_nontemporal_store(o, dst);
                        else *dst = o;
                    }
                } else {
                    // adjacent lanes on adjacent floats: an addition of MT floats per lane visits every cache line MT times
                    if (MT > 1) {
                        sl_lanes_meet();
                        *reinterpret_cast<TVec *>(swap_s + MT * lane) = o;
                        sl_lanes_meet();
                    }
#pragma unroll
                    for (int x = 0; x < MT; ++x) {
                        const float v = MT > 1 ? swap_s[16 * MT * kk + 16 * x + col] : o[0];
                        const int m = m0 + 16 * x + col;
                        if (!EDGE || (l < L && m < W)) atomic_add(A + l * W + m, v);
                    }
                }
            }
    };

    int last_row = 0;
    bool goes_on = false;   // the slice the run ends in goes on in the next run
    Stage st;
    if (r.chunk0 < c_end) issue(ch, st);
    for (int c = r.chunk0; c < c_end; ++c) {
        const int from = c == r.chunk0 ? r.step : 0, to = c == r_end.chunk0 ? r_end.step : ch.nsteps;
        const int ns = ch.nsteps, sl_base = ch.slice0, rowv = st.row;
        const uint64_t gm = ch.gend, sm = ch.send;
        // ---- stage: registers -> LDS; steps past the chunk have no child ----
        const bool live = lane < ns;
        auto row_at = [&](int x, uint32_t row) { return (uint32_t)(live ? x : kNoRow) * row; };
        if (SRC == SRC_LEAVES) {
            const int nl = ch.nleaves;
            sl_lanes_meet();
#pragma unroll
            for (int q = 0; q < 4; ++q) swap_s[64 * q + lane] = 64 * q + lane < nl ? st.v[q] : 0.f;   // place 255 is zero in a chunk of fewer leaves
            sl_lanes_meet();
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = swap_s[st.at >> 8 * q & 255];
            uint4 *dst = reinterpret_cast<uint4 *>(rec_s + 4 * lane);
            auto word = [&](float x) { return live ? __builtin_bit_cast(uint32_t, x) : 0u; };
            dst[0] = uint4{row_at(st.leaf.x, a.rowD), word(v[0]), row_at(st.leaf.y, a.rowD), word(v[1])};
            dst[1] = uint4{row_at(st.leaf.z, a.rowD), word(v[2]), row_at(st.leaf.w, a.rowD), word(v[3])};
        } else {
            sl_lanes_meet();
#pragma unroll
            for (int q = 0; q < 4; ++q)   // (steps before the run's first are not read)
                rec_s[4 * lane + q].off = row_at(st.f0 + q < st.f1 ? st.f0 + q - fbase : kNoRow, a.rowD);
            if (st.f0 + 1 >= st.f1) st.j.y = kNoRow;
            if (st.f0 + 2 >= st.f1) st.j.z = kNoRow;
            if (st.f0 + 3 >= st.f1) st.j.w = kNoRow;
        }
        reinterpret_cast<uint4 *>(coff_s)[lane] =
            uint4{row_at(st.j.x, a.rowC), row_at(st.j.y, a.rowC), row_at(st.j.z, a.rowC), row_at(st.j.w, a.rowC)};
        sl_lanes_meet();
        ch = chunks[c + 1];
        if (c + 1 < c_end) issue(ch, st);

        for (int b = from; b < to; b += U) {
            const uint32_t gb = SRC == SRC_LEAVES ? (uint32_t)(gm >> b) : 0xffffffffu, sb = (uint32_t)(sm >> b);
            Rec rec[U];
            uint32_t co[U];
            TVec d[U];
            CVec c[U];
#pragma unroll
            for (int u = 0; u < U; ++u) rec[u] = rec_s[4 * (b + u) + kk];
#pragma unroll
            for (int u = 0; u < U; ++u) co[u] = coff_s[4 * (b + u) + kk];
#pragma unroll
            for (int u = 0; u < U; ++u) d[u] = sl_gather<MT>(rowsD, rec[u].off + d_lane);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (SRC == SRC_ROWS || (gb >> u & 1)) c[u] = sl_gather<LT>(rowsC, co[u] + c_lane);
            uint32_t ge = gb;
            __asm__ volatile("" : "+s"(ge));   // tests of its own below: a bit kept over the batch costs more scalar instructions
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (SRC == SRC_LEAVES) {
#pragma unroll
                    for (int x = 0; x < MT; ++x) t[x] += rec[u].v * d[u][x];
                } else {
                    t = d[u];
                }
                if (SRC == SRC_ROWS || (ge >> u & 1)) {
                    multiply(t, c[u]);
                    if (SRC == SRC_LEAVES) {
#pragma unroll
                        for (int x = 0; x < MT; ++x) t[x] = 0.f;
                    }
                    if (sb >> u & 1) {
                        const int row = __builtin_amdgcn_readlane(rowv, sl - sl_base);
                        gather_sums(acc, tot);
                        clear(tot);
                        if (open) emit(row, std::integral_constant<int, ADD>{});
                        else if (a.stream) emit(row, std::integral_constant<int, STREAM>{});
                        else emit(row, std::integral_constant<int, STORE>{});
                        clear(acc);
                        open = false;
                        ++sl;
                    }
                }
            }
            if ((b + U) % SPAN == 0) {
                gather_sums(tot, acc);
                clear(acc);
            }
        }
        if (c + 1 == c_end) {
            // a group cut by the run's end is multiplied as far as it has come
            if (SRC == SRC_LEAVES && !(gm >> (to - 1) & 1)) multiply(t, sl_gather<LT>(rowsC, coff_s[4 * (to - 1) + kk] + c_lane));
            goes_on = !(sm >> (to - 1) & 1);
            last_row = __builtin_amdgcn_readlane(rowv, min(sl - sl_base, 63));
            gather_sums(acc, tot);
        }
    }
    if constexpr (RPB > 1) {
        sl_sum_runs<RPB, WPR, MT * LT>(reinterpret_cast<sl_floatx4 (&)[MT * LT]>(acc), goes_on, open && sl == slice0, lds.sum, state_s, wave, lane);
        if (MT > 1 || TURNED) __syncthreads();   // the sums have been read: their space is the staging regions again
    }
    if (goes_on) emit(last_row, std::integral_constant<int, ADD>{});
}

template <int SRC>
void dispatch_slice(const SliceArgs &a, const SliceTables &st, hipStream_t stream)
{
    auto go = [&](auto lt, auto mt, auto wl, auto wm) {
        constexpr int LT = decltype(lt)::value, MT = decltype(mt)::value, WL = decltype(wl)::value, WM = decltype(wm)::value;
        constexpr int RPB = NT / 64 / (WL * WM);
        const int blocks = (a.nruns + RPB - 1) / RPB;
        if (a.L != 16 * LT * WL || a.W != 16 * MT * WM) slice_kernel<LT, MT, WL, WM, SRC, true><<<blocks, NT, 0, stream>>>(a, st.d_runs, st.d_chunks);
        else slice_kernel<LT, MT, WL, WM, SRC, false><<<blocks, NT, 0, stream>>>(a, st.d_runs, st.d_chunks);
    };
    const SliceShape sh = slice_shape(a.L, a.W);
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    auto over_m = [&](auto lt, auto wl) {
        if (sh.mt == 1) go(lt, I1{}, wl, I1{});
        else if constexpr (decltype(lt)::value == 4) {
            if (sh.wm == 1) go(lt, I2{}, wl, I1{});
            else if (sh.mt == 2 && sh.wm == 2) go(lt, I2{}, wl, I2{});
            else if constexpr (decltype(wl)::value == 1) go(lt, I2{}, wl, I4{});
            else go(lt, I4{}, wl, I2{});
        } else {
            if (sh.mt == 2) go(lt, I2{}, wl, I1{});
            else if (sh.wm == 1) go(lt, I4{}, wl, I1{});
            else go(lt, I4{}, wl, I2{});
        }
    };
    if (sh.lt == 1) over_m(I1{}, I1{});
    else if (sh.lt == 2) over_m(I2{}, I1{});
    else if (sh.wl == 1) over_m(I4{}, I1{});
    else over_m(I4{}, I2{});
}

}  // namespace

SliceShape slice_shape(int64_t L, int64_t W)
{
    SliceShape s;
    if (L < 1 || L > 128 || W < 4 || W > 128 || W % 4 || (L > 16 && L % 4)) return s;   // the 16-byte (8-byte) pieces a lane reads and stores
    s.lt = L <= 16 ? 1 : L <= 32 ? 2 : 4;
    s.mt = W <= 16 ? 1 : W <= 32 || s.lt == 4 ? 2 : 4;   // eight tiles per wavefront at most
    s.wl = L > 64 ? 2 : 1;
    if (L > 64 && W > 64) s.mt = 4;   // sixteen, since four wavefronts make a workgroup (in workgroups of eight 128 x 128 took 1390 us for 1060)
    s.wm = W <= 16 * s.mt ? 1 : W <= 32 * s.mt ? 2 : 4;
    return s;
}

sc_status launch_slice(const sc_plan *p, Launcher &ln, const sc_csf_view *sp, const sc_dense_view &C, const sc_dense_view *D, const void *T,
                       int64_t W, void *out, const char *name)
{
    const SliceTables &st = p->slice;
    if (!st.d_runs) return SC_ERR_SCHED_UNSUPPORTED;
    SliceArgs a = {};
    a.nruns = st.nruns;
    a.leaf = st.d_leaf;
    a.at = st.d_at;
    a.gj = st.d_gj;
    a.first = st.d_first;
    a.crd1 = sp->crd[0];
    a.crd2 = sp->crd[1];
    a.nslices = (int32_t)p->nfib[0];
    a.vals = static_cast<const float *>(sp->vals);
    a.C = static_cast<const float *>(C.data);
    a.rowC = (uint32_t)(C.ld * 4);
    a.D = static_cast<const float *>(T ? T : D->data);
    a.rowD = (uint32_t)(T ? W * 4 : D->ld * 4);
    a.bytesC = (uint32_t)C.rows * a.rowC;   // (below 2 GiB: checked before anything is launched)
    a.bytesD = T ? kMostBytes : (uint32_t)D->rows * a.rowD;
    a.A = static_cast<float *>(out);
    a.L = (int32_t)C.cols;
    a.W = (int32_t)W;
    const int64_t children = T ? p->nfib[1] : p->nnz;
    a.stream = stores_past_caches(p->out_elems * 4, !p->zero_selective, p->nfib[0] * a.L * W * 4, (double)children / (double)std::max<int64_t>(p->nfib[0], 1), a.L, W, T != nullptr);
    ln.begin(name);
    if (T) dispatch_slice<SRC_ROWS>(a, st, ln.stream);
    else dispatch_slice<SRC_LEAVES>(a, st, ln.stream);
    ln.end();
    return ln.status;
}

}  // namespace sck
