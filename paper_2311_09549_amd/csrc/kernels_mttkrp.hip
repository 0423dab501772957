// Fused MTTKRP over steps: A(i,:) = sum over the fibers f of slice i of C(j_f,:) * t(f,:), t(f,:) = sum over the leaves of f of B * D(k,:),
// the Hadamard counterpart of the slice products (kernels_slice.hip), for rows of 64 and 128 bytes.  LG lanes hold a row, 16 bytes each; the
// G = 64 / LG lane groups of a wavefront take pieces of G fibers of a slice at a time, grouped by length, so that all of them end in the same
// step: a row of C is gathered once per group of pieces, with every lane in use, where a walk of each lane group for itself gathers under the mask of the fibers that end at every step.  A
// gather of 16 bytes per lane takes the L1 address path 16 cycles whatever its mask, and that path is what bounds these kernels.
// 20 M entries at rank 32: 182 us in the kernel over tiles and 157 so; the path is 0.92 busy, at 21 cycles per gather where the rows that come
// from the L2 (2 cycles a line) are counted in; at rank 16 174 and 136.
// A wavefront owns a run of steps; there is no barrier until its end.  The sum over a slice stays in registers, is added up over the lane groups where the
// slice ends, and stored; a slice cut by a run's end is added to the zeroed row atomically,
// after the runs of a workgroup that lie inside one slice have been added up in LDS.
#include "slice_common.h"

#include <type_traits>

namespace sck {

namespace {

struct MttkrpArgs {
    int32_t nruns, nslices;
    const uint32_t *leaf, *at;   // last coordinates, G per step; places of the values in the chunk (bytes)
    const int32_t *gj;           // G per group: coordinate of the row of C
    const int32_t *crd1;         // output row of every slice
    const void *vals, *C, *D;
    uint32_t rowC, rowD, bytesC, bytesD;
    void *A;
};

template <typename T, int LG>
__global__ void __launch_bounds__(NT, 4) mttkrp3_steps_kernel(MttkrpArgs a, const SliceRun *__restrict__ runs, const SliceChunk *__restrict__ chunks)
{
    constexpr int VEC = 16 / (int)sizeof(T), G = 64 / LG, R = LG * VEC, WAVES = NT / 64;
    constexpr int U = sizeof(T) == 4 ? 8 : 4;   // steps per batch: 3 M entries in fp64 52.7 us with eight, 40.6 with four; 20 M in fp32 168 and 176
    static_assert(G >= 4, "four places of a lane belong to one step");
    typedef T Vec __attribute__((ext_vector_type(VEC)));
    struct alignas(2 * sizeof(T)) Rec { uint32_t off; T v; };
    struct Own {                       // a wavefront's own staging region
        alignas(16) Rec rec[256];
        uint32_t coff[256];
        T swap[256];                   // the chunk's values while it is staged
    };
    union Lds {
        Own own[WAVES];
        Vec sum[2][64];                // after the runs: sums on their way to another wavefront
    };
    __shared__ Lds lds;
    __shared__ int state_s[WAVES];
    Own(&own)[WAVES] = lds.own;
    static_assert(sizeof(lds) + sizeof(state_s) <= mttkrp_steps_lds_bytes(sizeof(T)), "LDS the plan reports");

    const int wave = sl_uni(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int g = lane / LG;
    const uint32_t in_row = 16 * (lane % LG);
    const int run = (int)blockIdx.x * WAVES + wave;
    Rec *rec_s = own[wave].rec;
    uint32_t *coff_s = own[wave].coff;
    T *swap_s = own[wave].swap;
    const T *vals = static_cast<const T *>(a.vals);
    const __amdgpu_buffer_rsrc_t rowsC = sl_rows(a.C, a.bytesC), rowsD = sl_rows(a.D, a.bytesD);
    auto gather = [&](__amdgpu_buffer_rsrc_t rows, uint32_t off) { return __builtin_bit_cast(Vec, sl_gather<4>(rows, off + in_row)); };

    // a wavefront past the last run has no steps
    const SliceRun r = runs[min(run, a.nruns)], r_end = runs[min(run + 1, a.nruns)];
    const int c_end = r_end.chunk0 + (r_end.step > 0 ? 1 : 0);   // one past the last chunk of which this run has steps
    SliceChunk ch = chunks[r.chunk0];
    const int slice0 = ch.slice0 + __builtin_popcountll(ch.send & ((1ull << r.step) - 1));
    int sl = slice0;
    bool open = (r.flags & 1) != 0;   // the slice began in an earlier run

    // Global reads of a chunk's staging, issued a chunk ahead: a lane takes four places, 4 lane .. 4 lane + 3 (places past the chunk repeat its last ones).
    struct Stage {
        uint4 leaf;
        uint32_t at;
        int4 j;
        T v[4];
        int row;
    };
    auto issue = [&](const SliceChunk &c, Stage &s) {
        const int n = min(lane, c.nsteps * (G / 4) - 1), step = n / (G / 4);
        s.row = a.crd1[min(c.slice0 + lane, a.nslices - 1)];   // the output rows of the slices the chunk may complete
        s.leaf = *reinterpret_cast<const uint4 *>(a.leaf + (int64_t)c.step0 * G + 4 * n);
        s.at = a.at[(int64_t)c.step0 * (G / 4) + n];
        const int grp = min(__builtin_popcountll(c.gend & ((1ull << step) - 1)), c.ngroups - 1);
        s.j = *reinterpret_cast<const int4 *>(a.gj + (int64_t)(c.group0 + grp) * G + 4 * (n % (G / 4)));
#pragma unroll
        for (int q = 0; q < 4; ++q) s.v[q] = vals[c.leaf0 + min(64 * q + lane, c.nleaves - 1)];
    };

    // Sums of up to a batch of steps, and sums of those: shorter chains of additions (20 M entries: 2.2e-7 from the sum in double precision, where the
    // kernel over tiles is 3.1e-7).
    Vec t = {}, acc = {}, tot = {};
    // The sum over the lane groups, one element per lane.
    auto emit = [&](int row, bool add) {
        int ln = lane;
        __asm__ volatile("" : "+v"(ln));   // addresses are worked out here: kept over the loop they cost registers
        sl_lanes_meet();
        *reinterpret_cast<Vec *>(swap_s + VEC * ln) = acc + tot;
        sl_lanes_meet();
        T *A = static_cast<T *>(a.A) + (int64_t)row * R;
        if (ln < R) {
            T sum = swap_s[ln];
#pragma unroll
            for (int n = 1; n < G; ++n) sum += swap_s[n * R + ln];
            if (add) atomic_add(A + ln, sum);
            else A[ln] = sum;
        }
        acc = Vec{};
        tot = Vec{};
    };

    int last_row = 0;
    bool goes_on = false;   // the slice the run ends in goes on in the next run
    Stage st;
    if (r.chunk0 < c_end) issue(ch, st);
    for (int c = r.chunk0; c < c_end; ++c) {
        const int from = c == r.chunk0 ? r.step : 0, to = c == r_end.chunk0 ? r_end.step : ch.nsteps;
        const int places = ch.nsteps * G, nl = ch.nleaves, sl_base = ch.slice0, rowv = st.row;
        const uint64_t gm = ch.gend, sm = ch.send;
        // ---- stage: registers -> LDS; places past the chunk have no child ----
        sl_lanes_meet();
#pragma unroll
        for (int q = 0; q < 4; ++q) swap_s[64 * q + lane] = 64 * q + lane < nl ? st.v[q] : T(0);   // place 255 is zero in a chunk of fewer leaves
        sl_lanes_meet();
        const uint32_t leaf[4] = {st.leaf.x, st.leaf.y, st.leaf.z, st.leaf.w};
        T v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = swap_s[st.at >> 8 * q & 255];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool live = 4 * lane + q < places;
            Rec rec;
            rec.off = (uint32_t)(live ? (int)leaf[q] : kNoRow) * a.rowD;
            rec.v = live ? v[q] : T(0);
            rec_s[4 * lane + q] = rec;
        }
        reinterpret_cast<uint4 *>(coff_s)[lane] = uint4{(uint32_t)st.j.x * a.rowC, (uint32_t)st.j.y * a.rowC, (uint32_t)st.j.z * a.rowC, (uint32_t)st.j.w * a.rowC};
        sl_lanes_meet();
        if (from > 0 && !(gm >> (from - 1) & 1)) {
            // The run begins inside a group: a piece whose leaves all lie in the run before has no row in this one (its sum here is zero, and
            // zero times a row with an infinity is no number).
            int ln = lane, none = kNoRow;
            __asm__ volatile("" : "+v"(ln), "+s"(none));   // worked out here: kept over the loop it costs registers
            const int end = from + __builtin_ctzll(gm >> from), g = ln / LG;
            if (rec_s[G * from + g].off == none * a.rowD) coff_s[G * end + g] = coff_s[G * min(end, to - 1) + g] = none * a.rowC;
            sl_lanes_meet();
        }
        ch = chunks[c + 1];
        if (c + 1 < c_end) issue(ch, st);

        for (int b = from; b < to; b += U) {
            const uint32_t gb = (uint32_t)(gm >> b), sb = (uint32_t)(sm >> b);
            Rec rec[U];
            uint32_t co[U];
            Vec d[U], cv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) rec[u] = rec_s[G * (b + u) + g];
#pragma unroll
            for (int u = 0; u < U; ++u) co[u] = coff_s[G * (b + u) + g];
#pragma unroll
            for (int u = 0; u < U; ++u) d[u] = gather(rowsD, rec[u].off);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (gb >> u & 1) cv[u] = gather(rowsC, co[u]);
            uint32_t ge = gb;
            __asm__ volatile("" : "+s"(ge));   // tests of their own below: a bit kept over the batch costs more scalar instructions
#pragma unroll
            for (int u = 0; u < U; ++u) {
                t += rec[u].v * d[u];
                if (ge >> u & 1) {
                    acc += cv[u] * t;
                    t = Vec{};
                    if (sb >> u & 1) {
                        emit(__builtin_amdgcn_readlane(rowv, sl - sl_base), open);
                        open = false;
                        ++sl;
                    }
                }
            }
            tot += acc;
            acc = Vec{};
        }
        if (c + 1 == c_end) {
            // a group cut by the run's end is multiplied as far as it has come
            if (!(gm >> (to - 1) & 1)) acc += gather(rowsC, coff_s[G * (to - 1) + g]) * t;
            goes_on = !(sm >> (to - 1) & 1);
            last_row = __builtin_amdgcn_readlane(rowv, min(sl - sl_base, 63));
        }
    }
    acc += tot;
    tot = Vec{};
    sl_sum_runs<WAVES, 1, 1>(reinterpret_cast<Vec (&)[1]>(acc), goes_on, open && sl == slice0, lds.sum, state_s, wave, lane);
    __syncthreads();   // the sums have been read: their space is the staging regions again
    if (goes_on) emit(last_row, true);
}

}  // namespace

sc_status launch_mttkrp_steps(const sc_plan *p, Launcher &ln, const sc_csf_view *sp, const sc_dense_view *fac, void *out)
{
    const SliceTables &st = p->slice;
    if (!st.d_runs) return SC_ERR_SCHED_UNSUPPORTED;
    const uint32_t e = p->dtype == SC_F64 ? 8 : 4;
    MttkrpArgs a = {};
    a.nruns = st.nruns;
    a.nslices = (int32_t)p->nfib[0];
    a.leaf = st.d_leaf;
    a.at = st.d_at;
    a.gj = st.d_gj;
    a.crd1 = sp->crd[0];
    a.vals = sp->vals;
    a.C = fac[0].data;
    a.D = fac[1].data;
    a.rowC = (uint32_t)fac[0].ld * e;
    a.rowD = (uint32_t)fac[1].ld * e;
    a.bytesC = (uint32_t)fac[0].rows * a.rowC;   // (below 2 GiB: checked before anything is launched)
    a.bytesD = (uint32_t)fac[1].rows * a.rowD;
    a.A = out;
    const int blocks = (a.nruns + NT / 64 - 1) / (NT / 64);
    ln.begin("mttkrp3_fused");
    if (p->dtype == SC_F64) mttkrp3_steps_kernel<double, 8><<<blocks, NT, 0, ln.stream>>>(a, st.d_runs, st.d_chunks);
    else if (p->fcols[0] == 32) mttkrp3_steps_kernel<float, 8><<<blocks, NT, 0, ln.stream>>>(a, st.d_runs, st.d_chunks);
    else mttkrp3_steps_kernel<float, 4><<<blocks, NT, 0, ln.stream>>>(a, st.d_runs, st.d_chunks);
    ln.end();
    return ln.status;
}

}  // namespace sck
