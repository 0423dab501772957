// Order-4 TTM chain at 8 x 8 (L <= 16) on matrix cores, fp32, FUSED: the whole nest in one kernel without a barrier,
//     T1(f3, n)       = sum over the leaves of (i,j,k) fiber f3 of  B * E(p, n)
//     T2(f2, m, n)    = sum over the (i,j,k) fibers f3 of (i,j) fiber f2 of  D(k, m) * T1(f3, n)
//     A(i, l, m, n)   = sum over the (i,j) fibers f2 of slice i of  C(j, l) * T2(f2, m, n)
// (the shape of the second schedule of Table 2, kernel 5), as slice products are (kernels_slice.hip): a wavefront owns a run of steps, both
// temporaries stay in its registers and operands are gathered straight into them.
//
// The plan cuts (i,j) fibers into pieces of at most kChainPiece (i,j,k) fibers and takes four pieces of a slice at a time, a group, one for each
// 16 lanes kk; pieces with the same numbers of children and leaves go together.  A step is one leaf for each of the four.  Steps are taken in
// pairs: those of two children of one leaf each, or two of the steps of one child of several leaves (in each of the four pieces), so that
// which of the following happens is the same for the whole wavefront:
//   every pair              T1 += B * E(p, n)                       lanes 0 .. 7 of the 16 hold T1 of the pair's first step (child), lanes 8 .. 15 of
//                                                                   its second one: one gather for eight leaves
//   children end            T2(m, n) += D(k, m) * T1(n), twice      v_mfma_f32_4x4x1_16b_f32, four blocks for the outer product of 8 and 8 values of
//                                                                   each of four fibers: T1(4 nh + i) is copied to both halves, and of D(k, :), gathered once
//                                                                   for the pair, each product takes its two blocks of four lanes by the first operand's
//                                                                   broadcast; lane 4 (2 mh + nh) + i gets T2(4 mh + r, 4 nh + i), r = 0 .. 3
//   group ends              A(l, 4 mh + r, 4 nh + i) += T2 * C(j, l) four v_mfma_f32_16x16x4_f32, one per r: T2 lies in the registers as operand A
//                                                                   (row = lane of the 16, k = kk), the lane's value of the row of C is operand B
// so nothing passes through LDS from the leaves to the output.
//
// Bound by instruction issue: vector ALU 0.43 and matrix pipes 0.35 of the cycles at 3.6 wavefronts per SIMD, L1 address path 0.68.  Without the gathers 452
// us, without the products of group ends as well 340.  Repeated calls, 50 M entries at 8 x 8 x 8, 921 us in the kernel over tiles that ran before
// (both temporaries in LDS, three barriers per tile) and 550 now; a gather and a test per step and child, without the pairs, 605; rows of D gathered
// only where children end 560.
#include "slice_common.h"

#include <type_traits>

namespace sck {

namespace {

struct ChainArgs {
    int32_t nruns, nslices;
    const uint32_t *leaf, *at;   // 4 last coordinates per step, 4 places of the value in the chunk (bytes)
    const int32_t *gk;           // 4 per child group: coordinate of the row of D
    const int32_t *gj;           // 4 per group: coordinate of the row of C
    const int32_t *crd1;         // output row of every slice
    const float *vals;
    const float *C, *D, *E;
    uint32_t rowC, rowD, rowE, bytesC, bytesD, bytesE;
    float *A;
    int32_t L;
};

constexpr int CH_W = 64;         // elements (m, n) of a row of T2
constexpr int CH_U = kChainBatch / 2;   // pairs of steps per batch

// SMALL: every factor has less than 2^24 - 1 rows of at most 256 bytes, so that a row's offset is a product of 24 bits
template <bool SMALL>
__global__ void __launch_bounds__(NT, 4) chain4_kernel(ChainArgs a, const SliceRun *__restrict__ runs, const SliceChunk *__restrict__ chunks,
                                                       const ChainChunk *__restrict__ kids)
{
    constexpr int WAVES = NT / 64, U = CH_U;
    struct alignas(8) Rec { uint32_t off; float v; };
    struct Own {               // a wavefront's own staging region
        alignas(16) Rec rec[256];
        uint32_t doff[256];       // offsets of the rows of D ...
        uint32_t coff[256];       // ... and of C, [pair][kk][step of the pair]
        float swap[256];       // the chunk's values while it is staged; a row on its way to atomic additions
    };
    union Lds {
        Own own[WAVES];
        sl_floatx4 sum[2][4 * 64];   // after the runs: sums on their way to another wavefront
    };
    __shared__ Lds lds;
    __shared__ int state_s[WAVES];
    static_assert(sizeof(Lds) + sizeof(state_s) <= kChainLdsBytes, "LDS the plan reports");

    const int wave = sl_uni(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int kk = lane / 16, col = lane % 16;
    const int run = (int)blockIdx.x * WAVES + wave;
    Rec *rec_s = lds.own[wave].rec;
    uint32_t *doff_s = lds.own[wave].doff, *coff_s = lds.own[wave].coff;
    float *swap_s = lds.own[wave].swap;
    const int L = a.L;
    // Of a pair of steps lanes 0 .. 7 of the 16 gather for the first one, lanes 8 .. 15 for the second: the eight values of a row of E, whose
    // products are then copied to the other eight; of D blocks of four lanes by turns, which the first operand's broadcast serves.
    const int e_at = 4 * (col / 8) + kk, d_at = 4 * (col / 4 % 2) + kk;
    const uint32_t e_lane = 4 * (col % 8), d_lane = 4 * (4 * (col / 8) + col % 4), c_lane = 4 * min(col, L - 1);
    const __amdgpu_buffer_rsrc_t rowsC = sl_rows(a.C, a.bytesC), rowsD = sl_rows(a.D, a.bytesD), rowsE = sl_rows(a.E, a.bytesE);

    // a wavefront past the last run has no steps
    const SliceRun r = runs[min(run, a.nruns)], r_end = runs[min(run + 1, a.nruns)];
    const int c_end = r_end.chunk0 + (r_end.step > 0 ? 1 : 0);   // one past the last chunk of which this run has steps
    SliceChunk ch = chunks[r.chunk0];
    ChainChunk kc = kids[r.chunk0];
    const int slice0 = ch.slice0 + __builtin_popcountll(ch.send & ((1ull << r.step) - 1));
    int sl = slice0;
    bool open = (r.flags & 1) != 0;   // the slice began in an earlier run

    // Global reads of a chunk's staging: lane n takes step n (those past the chunk repeat its last one) and the children and the group that
    // step belongs to.  They are issued a chunk ahead and land while the one before is worked on.
    struct Stage {
        uint4 leaf;
        uint32_t at;
        int4 k, j;
        float v[4];
        int row;
    };
    auto before = [](uint64_t bits) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0)); };
    auto issue = [&](const SliceChunk &c, const ChainChunk &k, Stage &s) {
        const int n = min(lane, c.nsteps - 1);
        s.row = a.crd1[min(c.slice0 + lane, a.nslices - 1)];   // the output rows of the slices the chunk may complete
        s.leaf = reinterpret_cast<const uint4 *>(a.leaf)[c.step0 + n];
        s.at = a.at[c.step0 + n];
        s.k = reinterpret_cast<const int4 *>(a.gk)[2 * (k.kid0 + min(before(k.kend), k.nkids - 1)) + lane % 2];
        s.j = reinterpret_cast<const int4 *>(a.gj)[c.group0 + min(before(c.gend), c.ngroups - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) s.v[q] = a.vals[c.leaf0 + min(64 * q + lane, c.nleaves - 1)];
    };

    float t1 = 0.f;
    sl_floatx4 t2 = {0.f, 0.f, 0.f, 0.f};
    // Sums over a batch, and sums of those.  Distance from the sum in double precision, 50 M entries on a power law and 3 M uniform ones: one chain over a
    // run 5.1e-7 (kernel over tiles 2.3e-7); sums over a chunk 2.1e-7 and 2.3e-7 (1.6e-7); over a batch, 1 % slower, 2.3e-7 and 1.5e-7.
    sl_floatx4 acc[4], tot[4];   // acc[r][q] = A(l = col, m = 4 (kk / 2) + r, n = 4 (kk % 2) + q)
    auto clear = [](sl_floatx4 (&v)[4]) {
        for (sl_floatx4 &e : v) e = sl_floatx4{0.f, 0.f, 0.f, 0.f};
    };
    clear(acc);
    clear(tot);
    // the t1 of the first (second) step of a pair for all 16 lanes
    auto first = [](float x) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, x), __builtin_bit_cast(int, x), 0x128, 0xf, 0xc, false)); };
    auto second = [](float x) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, x), __builtin_bit_cast(int, x), 0x128, 0xf, 0x3, false)); };
    auto group = [&](float c) {
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(t2[x], c, acc[x], 0, 0, 0);
        t2 = sl_floatx4{0.f, 0.f, 0.f, 0.f};
    };
    auto emit = [&](int row, bool add) {
        int ln = lane;
        __asm__ volatile("" : "+v"(ln));   // addresses are worked out here: kept over the loop they cost registers
        const int kk = ln / 16, col = ln % 16;
        float *A = a.A + (int64_t)row * L * CH_W;
        if (!add) {
            float *dst = A + col * CH_W + 32 * (kk / 2) + 4 * (kk % 2);
            if (col < L)
#pragma unroll
                for (int x = 0; x < 4; ++x) *reinterpret_cast<sl_floatx4 *>(dst + 8 * x) = acc[x];
            return;
        }
        float *dst = A + kk * CH_W + 32 * (col / 8) + col % 8;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            // adjacent lanes on adjacent floats: the four of a lane one after the other visit every cache line four times
            sl_lanes_meet();
            *reinterpret_cast<sl_floatx4 *>(swap_s + 16 * col + 4 * kk) = acc[x];
            sl_lanes_meet();
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * q + kk < L) atomic_add(dst + 4 * q * CH_W + 8 * x, swap_s[64 * q + ln]);
        }
    };

    int last_row = 0;
    bool goes_on = false;   // the slice the run ends in goes on in the next run
    Stage st;
    if (r.chunk0 < c_end) issue(ch, kc, st);
    for (int c = r.chunk0; c < c_end; ++c) {
        const int from = c == r.chunk0 ? r.step : 0, to = c == r_end.chunk0 ? r_end.step : ch.nsteps;
        const int nl = ch.nleaves, sl_base = ch.slice0, rowv = st.row;
        const uint64_t km = kc.kend, gm = ch.gend, sm = ch.send;
        // ---- stage: registers -> LDS (lanes past the chunk's steps write what is not read) ----
        auto row_at = [&](uint32_t x, uint32_t row) { return SMALL ? (x & 0xffffffu) * (row & 0xffffffu) : x * row; };
        sl_lanes_meet();
#pragma unroll
        for (int q = 0; q < 4; ++q) swap_s[64 * q + lane] = q == 3 && lane == 63 && nl < 256 ? 0.f : st.v[q];   // place 255 is zero in a chunk of fewer leaves
        sl_lanes_meet();
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = swap_s[st.at >> 8 * q & 255];
        auto word = [](float x) { return __builtin_bit_cast(uint32_t, x); };
        uint4 *dst = reinterpret_cast<uint4 *>(rec_s + 4 * lane);
        dst[0] = uint4{row_at(st.leaf.x, a.rowE), word(v[0]), row_at(st.leaf.y, a.rowE), word(v[1])};
        dst[1] = uint4{row_at(st.leaf.z, a.rowE), word(v[2]), row_at(st.leaf.w, a.rowE), word(v[3])};
        reinterpret_cast<uint4 *>(doff_s)[lane] = uint4{row_at(st.k.x, a.rowD), row_at(st.k.y, a.rowD), row_at(st.k.z, a.rowD), row_at(st.k.w, a.rowD)};
        uint32_t *co = coff_s + 8 * (lane / 2) + lane % 2;
        co[0] = row_at(st.j.x, a.rowC);
        co[2] = row_at(st.j.y, a.rowC);
        co[4] = row_at(st.j.z, a.rowC);
        co[6] = row_at(st.j.w, a.rowC);
        sl_lanes_meet();
        if (from > 0 && !(gm >> (from - 1) & 1)) {
            // The run begins inside a group: a child whose leaves (a piece whose children) all lie in the run before has no row in this one (its sum
            // here is zero, and zero times a row with an infinity is no number).
            int ln = lane, none = kNoRow;
            __asm__ volatile("" : "+v"(ln), "+s"(none));   // worked out here: kept over the loop it costs registers
            const int kk = ln / 16, col = ln % 16, last = min(from + __builtin_ctzll(gm >> from), to - 1);
            const uint32_t no_leaf = row_at(none, a.rowE);
            bool any = false;
#pragma clang loop unroll(disable)
            for (int s = from + col; s <= last; s += 16) any |= rec_s[4 * s + kk].off != no_leaf;
            if (!(__ballot(any) >> 16 * kk & 0xffff)) coff_s[8 * (last / 2) + 2 * kk + last % 2] = row_at(none, a.rowC);
            if (!(km >> (from - 1) & 1) && col < 2 && rec_s[4 * (from + col) + kk].off == no_leaf)
                doff_s[4 * (min(from + __builtin_ctzll(km >> from) - 1, to - 2) + col) + kk] = row_at(none, a.rowD);   // (in the pair where they end)
            sl_lanes_meet();
        }
        ch = chunks[c + 1];
        kc = kids[c + 1];
        if (c + 1 < c_end) issue(ch, kc, st);

        for (int b = from; b < to; b += 2 * U) {
            const uint32_t kb = (uint32_t)(km >> b), gb = (uint32_t)(gm >> b), sb = (uint32_t)(sm >> b);
            Rec rec[U];
            uint32_t dof[U];
            float e[U], d[U], cv[2 * U];
#pragma unroll
            for (int u = 0; u < U; ++u) rec[u] = rec_s[4 * (b + 2 * u) + e_at];
#pragma unroll
            for (int u = 0; u < U; ++u) dof[u] = doff_s[4 * (b + 2 * u) + d_at];
#pragma unroll
            for (int u = 0; u < U; ++u) e[u] = sl_gather<1>(rowsE, rec[u].off + e_lane)[0];
#pragma unroll
            for (int u = 0; u < U; ++u) d[u] = sl_gather<1>(rowsD, dof[u] + d_lane)[0];   // (also where no child ends: a branch each takes longer, 560 us for 547)
            const uint32_t *co = coff_s + 4 * b + 2 * kk;
#pragma unroll
            for (int u = 0; u < 2 * U; ++u)
                if (gb >> u & 1) cv[u] = sl_gather<1>(rowsC, co[4 * (u - u % 2) + u % 2] + c_lane)[0];
            uint32_t ke = kb, ge = gb;
            __asm__ volatile("" : "+s"(ke), "+s"(ge));   // tests of their own below: a bit kept over the batch costs more scalar instructions
            auto group_ends = [&](int u) {
                group(cv[u]);
                if (sb >> u & 1) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) acc[x] += tot[x];
                    clear(tot);
                    emit(__builtin_amdgcn_readlane(rowv, sl - sl_base), open);
                    clear(acc);
                    open = false;
                    ++sl;
                }
            };
#pragma unroll
            for (int u = 0; u < U; ++u) {
                t1 += rec[u].v * e[u];
                if (ke >> (2 * u + 1) & 1) {
                    const float ta = first(t1), tb = second(t1);
                    t1 = 0.f;
                    t2 = __builtin_amdgcn_mfma_f32_4x4x1f32(d[u], ta, t2, 1, 0, 0);
                    if (ge >> 2 * u & 1) group_ends(2 * u);
                    t2 = __builtin_amdgcn_mfma_f32_4x4x1f32(d[u], tb, t2, 1, 1, 0);
                    if (ge >> (2 * u + 1) & 1) group_ends(2 * u + 1);
                }
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) tot[x] += acc[x];
            clear(acc);
        }
        if (c + 1 == c_end) {
            // children and a group cut by the run's end are multiplied as far as they have come
            const int p = to - 2;
            if (!(km >> (to - 1) & 1)) {
                const float d = sl_gather<1>(rowsD, doff_s[4 * p + d_at] + d_lane)[0];
                t2 = __builtin_amdgcn_mfma_f32_4x4x1f32(d, first(t1), t2, 1, 0, 0);
                t2 = __builtin_amdgcn_mfma_f32_4x4x1f32(d, second(t1), t2, 1, 1, 0);
            }
            if (!(gm >> (to - 1) & 1)) group(sl_gather<1>(rowsC, coff_s[4 * p + 2 * kk + 1] + c_lane)[0]);
            goes_on = !(sm >> (to - 1) & 1);
            last_row = __builtin_amdgcn_readlane(rowv, min(sl - sl_base, 63));
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[x] += tot[x];
        }
    }
    sl_sum_runs<WAVES, 1, 4>(acc, goes_on, open && sl == slice0, lds.sum, state_s, wave, lane);
    __syncthreads();   // the sums have been read: their space is the staging regions again
    if (goes_on) emit(last_row, true);
}

}  // namespace

sc_status launch_chain4(const sc_plan *p, Launcher &ln, const sc_csf_view *sp, const sc_dense_view *fac, void *out)
{
    const SliceTables &st = p->slice;
    if (!st.d_runs) return SC_ERR_SCHED_UNSUPPORTED;
    ChainArgs a = {};
    a.nruns = st.nruns;
    a.nslices = (int32_t)p->nfib[0];
    a.leaf = st.d_leaf;
    a.at = st.d_at;
    a.gk = st.d_gk;
    a.gj = st.d_gj;
    a.crd1 = sp->crd[0];
    a.vals = static_cast<const float *>(sp->vals);
    auto matrix = [](const sc_dense_view &f, const float *&data, uint32_t &row, uint32_t &bytes) {   // (below 2 GiB: checked before anything is launched)
        data = static_cast<const float *>(f.data);
        row = (uint32_t)(f.ld * 4);
        bytes = (uint32_t)f.rows * row;
    };
    matrix(fac[0], a.C, a.rowC, a.bytesC);
    matrix(fac[1], a.D, a.rowD, a.bytesD);
    matrix(fac[2], a.E, a.rowE, a.bytesE);
    a.A = static_cast<float *>(out);
    a.L = (int32_t)p->fcols[0];
    ln.begin("ttmc4_fused_mfma");
    bool small = true;
    for (int s = 0; s < 3; ++s) small = small && fac[s].rows < (1 << 24) - 1 && fac[s].ld <= 64;
    const int blocks = (a.nruns + NT / 64 - 1) / (NT / 64);
    if (small) chain4_kernel<true><<<blocks, NT, 0, ln.stream>>>(a, st.d_runs, st.d_chunks, st.d_kids);
    else chain4_kernel<false><<<blocks, NT, 0, ln.stream>>>(a, st.d_runs, st.d_chunks, st.d_kids);
    ln.end();
    return ln.status;
}

}  // namespace sck
