// All-mode TTMC, kernel 5 of Table 2 (the running example of Sections 1 and 3):
//     A(l,m,n) = sum_ijk B(i,j,k) * C(i,l) * D(j,m) * E(k,n)
// under the three schedules Table 2 lists for it.  The output carries no sparse index, so whatever
// the nest produces per slice (or per fiber) has to be reduced over the whole grid; that last
// contraction is what this file adds.  The sparse part reuses the order-3 TTM chain
//     S(i,m,n) = sum_jk B(i,j,k) * D(j,m) * E(k,n)
// of the library (an inner plan over the same tensor with factors D and E):
//
//   schedule 2 (default)  i,n < T_m; j' < t; k': t += B E, m: T_m += t D >, m,l: A += T_m C >
//                         inner plan FUSED (t and T_m on chip) or FISSIONED (t(i,j,n) in the
//                         workspace), then mode0_reduce: A(l,:) += C(i,l) * S(i,:)
//   schedule 3            i,m,n < t; j',k': t += B D E, l: A += t C >
//                         inner plan LINEAR (the unfactored nest per slice), then mode0_reduce
//   schedule 1            i,j',n < t; k': t += B E, m,l: A += t C D >
//                         leaf traversal of the inner plan (t(i,j,:) per fiber in the workspace), then
//                         fiber_reduce: A(l,m,n) += C(i,l) * D(j,m) * t(f,n) over all fibers
//
// Both reductions are deterministic: a workgroup sums a contiguous chunk of slices (fibers) into an
// L x (M N) tile in registers and stores it in its own slot of the workspace; sum_partials adds the
// slots in chunk order.  The reduction over i is a dense (L x I) * (I x MN) product with I large:
// 2 L flops per 4-byte element of S read.  In fp32 with L in {16, 32, 64, 128} and M N a multiple of 64 it runs
// on the matrix cores with all of L per wavefront, so that S is read once whatever L is; the other cases
// (fp64, other ranks) run on the vector ALUs, a thread per column with 16 values of l in registers.
#include "device_common.h"

#include <type_traits>

namespace sck {

namespace {

constexpr int KB_L = 16;     // output slabs (values of l) one thread accumulates
constexpr int KR_ROWS = 64;  // rows of C staged per pass of mode0_reduce

struct K5Args {
    const void *C;
    int64_t ldC;
    const void *D;
    int64_t ldD;
    const void *S;          // mode0_reduce: I x MN, row-major; fiber_reduce: t rows, F x N
    const int32_t *crd1, *pos2, *crd2;   // fiber_reduce: slices and fibers of the tensor
    void *partials;         // nchunks x L x MN
    int64_t rows;           // I (mode0_reduce) or F (fiber_reduce)
    int32_t nslices;        // fiber_reduce: non-empty slices
    int32_t L, M, N, MN;
    int32_t chunk;          // rows (slices / fibers) per workgroup
};

// partial(b, l, c) = sum_{i in chunk b} C(i,l) * S(i,c); thread = column c, KB_L values of l in registers
template <typename T>
__global__ void __launch_bounds__(NT) mode0_reduce_kernel(K5Args a)
{
    __shared__ T c_s[KR_ROWS * KB_L];
    const int tid = threadIdx.x;
    const int c = blockIdx.y * NT + tid;
    const int l0 = blockIdx.z * KB_L;
    const int nl = min(KB_L, a.L - l0);
    const int64_t r0 = (int64_t)blockIdx.x * a.chunk, r1 = min(r0 + a.chunk, a.rows);
    const T *C = static_cast<const T *>(a.C);
    const T *S = static_cast<const T *>(a.S);
    T acc[KB_L];
#pragma unroll
    for (int l = 0; l < KB_L; ++l) acc[l] = T(0);
    for (int64_t rb = r0; rb < r1; rb += KR_ROWS) {
        const int nr = (int)min<int64_t>(KR_ROWS, r1 - rb);
        __syncthreads();
        for (int e = tid; e < KR_ROWS * KB_L; e += NT) {
            const int r = e / KB_L, l = e % KB_L;
            c_s[e] = (r < nr && l < nl) ? C[(rb + r) * a.ldC + l0 + l] : T(0);
        }
        __syncthreads();
        if (c < a.MN) {
            for (int r = 0; r < nr; ++r) {
                const T s = S[(rb + r) * (int64_t)a.MN + c];
#pragma unroll
                for (int l = 0; l < KB_L; ++l) acc[l] += c_s[r * KB_L + l] * s;
            }
        }
    }
    if (c < a.MN) {
        T *P = static_cast<T *>(a.partials) + (int64_t)blockIdx.x * a.L * a.MN;
        for (int l = 0; l < nl; ++l) P[(int64_t)(l0 + l) * a.MN + c] = acc[l];
    }
}

// The same partial sums on the matrix cores, fp32, L = 16 LT in {16, 32, 64, 128}, M N a multiple of 64: a wavefront takes all of L
// for 16 X columns (X = 4 or 1); four slices per v_mfma_f32_16x16x4_f32 with C^T as operand A (l along the rows) and S
// as operand B, both straight from global memory.  Which l and which column a tile's rows and columns stand for is free, so
// a lane reads 4 X adjacent bytes of a row of S (one column in each of the wavefront's X column tiles) and up to 16 of a row
// of C (one l in each of four l tiles): three loads per 4 LT MFMAs at L = 128 and X = 4.  With 4-byte loads, nine per LT MFMAs, 40,000 slices
// at 128 x 128 x 128 took 2606 us = 66 TFLOP/s, where the fp32 matrix rate of a large library product is 149; 1532 us = 110
// now.  The reads of the next UK steps are in flight while this batch is multiplied; the wavefronts of a workgroup read
// the same rows of C.
// X = 4 reads S and C with the fewest instructions; where it leaves most SIMDs without a wavefront, X = 1 has four
// times the wavefronts and a quarter of the chain of MFMAs in each.  Whole calls, 100,000 nonzeros in 4,000 slices (63 chunks): 128 x 16 x 16
// 33.2 us with X = 4, 26.7 with X = 1; 64 x 16 x 16 26.3 and 23.7.
typedef float k5_floatx4 __attribute__((ext_vector_type(4)));
template <int LT, int X>
__global__ void __launch_bounds__(NT, 2) mode0_reduce_mfma_kernel(K5Args a)
{
    typedef float SVec __attribute__((ext_vector_type(X)));
    constexpr int UK = LT * X >= 32 ? 2 : 4;   // steps of four slices per batch of reads
    constexpr int CW = LT < 4 ? LT : 4;    // adjacent values of l a lane reads at once ...
    constexpr int CN = LT / CW;            // ... in CN pieces, 16 CW values of l apart
    const int tid = threadIdx.x;
    const int wave = tid / 64, lane = tid % 64, kk = lane / 16, col = lane % 16;
    const int c = ((int)blockIdx.y * ((int)blockDim.x / 64) + wave) * 16 * X + X * col;   // < M N: the launch has M N / (16 X) wavefronts along y
    const int64_t r0 = (int64_t)blockIdx.x * a.chunk, r1 = min(r0 + a.chunk, a.rows);
    const float *C = static_cast<const float *>(a.C) + CW * col;
    const float *S = static_cast<const float *>(a.S) + c;
    struct Batch {
        SVec s[UK];
        Pack<float, CW> v[UK][CN];
    };
    auto load = [&](Batch &b, int64_t rb) {
#pragma unroll
        for (int u = 0; u < UK; ++u) {
            const int64_t row = rb + 4 * u + kk;
            b.s[u] = *reinterpret_cast<const SVec *>(S + row * a.MN);
#pragma unroll
            for (int h = 0; h < CN; ++h) b.v[u][h] = *reinterpret_cast<const Pack<float, CW> *>(C + row * a.ldC + 16 * CW * h);
        }
    };
    k5_floatx4 acc[LT][X];
#pragma unroll
    for (int lt = 0; lt < LT; ++lt)
#pragma unroll
        for (int x = 0; x < X; ++x) acc[lt][x] = k5_floatx4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](const SVec &s, const Pack<float, CW> (&v)[CN]) {
#pragma unroll
        for (int lt = 0; lt < LT; ++lt)
#pragma unroll
            for (int x = 0; x < X; ++x)
                acc[lt][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[lt / CW].v[lt % CW], s[x], acc[lt][x], 0, 0, 0);
    };
    const int64_t nfull = (r1 - r0) / (4 * UK);   // batches without a row past the chunk
    if (nfull > 0) {
        Batch cur, next;
        load(cur, r0);
        for (int64_t b = 0; b < nfull; ++b) {
            load(next, r0 + min(b + 1, nfull - 1) * (4 * UK));
            __builtin_amdgcn_sched_barrier(0);   // the compiler would otherwise sink these reads below the products
#pragma unroll
            for (int u = 0; u < UK; ++u) step(cur.s[u], cur.v[u]);
            cur = next;
        }
    }
    for (int64_t rb = r0 + nfull * (4 * UK); rb < r1; rb += 4) {
        const int64_t row = min(rb + kk, r1 - 1);   // lanes past the chunk read its last slice and are zeroed
        const bool ok = rb + kk < r1;
        SVec s = *reinterpret_cast<const SVec *>(S + row * a.MN);
        Pack<float, CW> v[CN];
#pragma unroll
        for (int x = 0; x < X; ++x) s[x] = ok ? s[x] : 0.f;
#pragma unroll
        for (int h = 0; h < CN; ++h) {
            v[h] = *reinterpret_cast<const Pack<float, CW> *>(C + row * a.ldC + 16 * CW * h);
#pragma unroll
            for (int i = 0; i < CW; ++i) v[h].v[i] = ok ? v[h].v[i] : 0.f;
        }
        step(s, v);
    }
    // acc[lt][x][r] = partial(l = 16 CW (lt / CW) + CW (4 kk + r) + lt % CW, column c + x)
    float *P = static_cast<float *>(a.partials) + (int64_t)blockIdx.x * a.L * a.MN + c;
#pragma unroll
    for (int lt = 0; lt < LT; ++lt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int l = 16 * CW * (lt / CW) + CW * (4 * kk + r) + lt % CW;
            SVec o;
#pragma unroll
            for (int x = 0; x < X; ++x) o[x] = acc[lt][x][r];
            *reinterpret_cast<SVec *>(P + (int64_t)l * a.MN) = o;
        }
}

// The same partial sums from products of 16 bits: a value of 24 bits is the exact sum of three of 8, x = h + m + l, each of them a
// bf16 (h the nearest to x, m to x - h, l what is left), and a product of two of them is exact in fp32.  Of the nine
// products of parts the three below 2^-26 of the whole, m l, l m and l l, are left out; the other six are added in fp32, the small ones
// first, by v_mfma_f32_16x16x32_bf16, which takes 32 slices at 16 times the fp32 rate.
// C is split once by a launch of its own into rows of eight slices (k5_split_kernel), so that a lane reads operand A, eight slices of one l, with
// one 16-byte load per part; S is read as it is, eight slices of four columns per lane, and split in registers: it passes once.
// Parts hold values from 2^-109 on, below which the last bits are lost, to 2^127, past which h may be infinite.  A step of which C or S has smaller ones
// (C's are marked by the launch that splits it) is left for products in fp32 after the others; where a sum turns out not to be finite the whole chunk is
// added up again in fp32 (k5_again): infinities, NaN, values past the largest bf16 and small ones give what the fp32 form gives, in about five times its time.
// The tests for it take 1 to 5 % of the reduction (64 x 64 x 64 154 us without, 158 with them; 128 x 64 x 64 222 and 234; 128 x 128 x 128 even).
// Repeated calls, the reduction alone, 40,000 slices, fp32 and this form: 128 x 128 x 128 1398 and 810 us (S alone takes 450), 128 x 64 x 64 372 and 234,
// 64 x 64 x 64 202 and 158.  Error against double precision 1.31e-6 and 0.74e-6, 6.4e-7 and 4.1e-7, 6.4e-7 and 2.0e-7; of inputs of one sign 4.2e-7 and
// 1.4e-7, 1.3e-7 and 0.8e-7, 1.3e-7 and 0.6e-7; 3 million slices at 128 x 16 x 16, chunks of 5,900, 1.36e-6 and 1.16e-6, of one sign 1.2e-7 and 1.0e-7.
// (Where all inputs are alike every slice is rounded the same way, and either form may be ahead: at ten sizes, 995 to a million slices at L = 64 and 128, the
// fp32 form is 1.3e-7 to 2.8e-5 off and this one 0.2e-7 to 2.9e-6, in three of them further than fp32.  Of random inputs and of one sign it is ahead at all ten.)
// At L = 64 the six products of a step are added up apart from the sum they go to; at L = 128, whose registers are
// full, that took longer (942 us for 765), and shorter chunks serve instead (plan_ttmc_all).
constexpr int K5_K = 32;   // slices per step
typedef __bf16 k5_bf16 __attribute__((ext_vector_type(8)));

// whether some of N values are not zero but smaller than 2^-109
template <int N>
__device__ __forceinline__ bool k5_small(const float (&x)[N])
{
    uint32_t least = 0xffffffffu;
#pragma unroll
    for (int j = 0; j < N; ++j) least = min(least, (__builtin_bit_cast(uint32_t, x[j]) << 1) - 1);   // |x| doubled as an integer, less one: zero is the largest
    return least < (18u << 24) - 1;
}

// the nearest bf16 of a (low half) and b
__device__ __forceinline__ uint32_t k5_pack(float a, float b)
{
    typedef float F2 __attribute__((ext_vector_type(2)));
    typedef __bf16 B2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(F2{a, b}, B2));
}

// the three parts of eight values
__device__ __forceinline__ void k5_parts(const float (&x)[8], uint4 (&part)[3])
{
    float r[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = x[j];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = k5_pack(r[2 * j], r[2 * j + 1]);
        part[p] = uint4{w[0], w[1], w[2], w[3]};
        if (p < 2)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                r[2 * j] -= __builtin_bit_cast(float, w[j] << 16);
                r[2 * j + 1] -= __builtin_bit_cast(float, w[j] & 0xffff0000u);
            }
    }
}

// C3[part][slices / 8][l][8], slices up to a multiple of 32; slices past the last are zero.  L is 64 or 128, so that a workgroup's values are those of a step or half of one, and there
// are no threads past the last: marks[workgroup] says whether some are too small for the parts.
__global__ void __launch_bounds__(NT) k5_split_kernel(const float *__restrict__ C, int64_t ldC, int64_t rows, int L, int64_t groups, uint4 *__restrict__ C3,
                                                      uint32_t *__restrict__ marks)
{
    const int64_t n = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int64_t g = n / L;
    const int l = (int)(n % L);
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = 8 * g + j < rows ? C[(8 * g + j) * ldC + l] : 0.f;
    const int small = __syncthreads_or(k5_small(x));
    if (threadIdx.x == 0) marks[blockIdx.x] = small;
    uint4 part[3];
    k5_parts(x, part);
#pragma unroll
    for (int p = 0; p < 3; ++p) C3[(int64_t)p * groups * L + n] = part[p];
}

// whether a step is left for fp32: the values of S that the lane has, and the marks of C
template <int LT>
__device__ __forceinline__ bool k5_leave(const k5_floatx4 (&raw)[8], const uint32_t *marks, int64_t step)
{
    uint32_t marked = marks[step * (LT / 4)];
    if (LT == 8) marked |= marks[step * (LT / 4) + 1];
    float least = 1.f;
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int j = 0; j < 8; j += 2) __asm__("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(least) : "v"(raw[j][x]), "v"(raw[j + 1][x]));
    bool some = least < 0x1p-109f;
    if (__any(some)) {   // zeros, which slices without an entry are full of, or others
        float v[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) v[j] = raw[j / 4][j % 4];
        some = k5_small(v);
    }
    return marked || __any(some);
}

// Adds the steps of a chunk that were left (all) to (as) what is stored, an l tile at a time: four slices per v_mfma_f32_16x16x4_f32, whose sums lie as
// those of the kernel below.
template <int LT>
__device__ __forceinline__ void k5_again(const K5Args &a, int64_t r0, int64_t r1, int c, int kk, int col, const uint32_t *marks, bool all)
{
    const float *S = static_cast<const float *>(a.S) + c;
#pragma clang loop unroll(disable)
    for (int l = 0; l < 16 * LT; l += 16) {
        float *P = static_cast<float *>(a.partials) + ((int64_t)blockIdx.x * a.L + l + 4 * kk) * a.MN + c;
        const float *C = static_cast<const float *>(a.C) + l + col;
        k5_floatx4 sum[4] = {};
        if (!all)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const k5_floatx4 was = *reinterpret_cast<const k5_floatx4 *>(P + (int64_t)q * a.MN);
#pragma unroll
                for (int x = 0; x < 4; ++x) sum[x][q] = was[x];
            }
#pragma clang loop unroll(disable)
        for (int64_t r = r0; r < r1; r += K5_K) {
            if (!all) {
                k5_floatx4 raw[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) raw[j] = *reinterpret_cast<const k5_floatx4 *>(S + min(r + 8 * kk + j, a.rows - 1) * a.MN);
                if (!k5_leave<LT>(raw, marks, r / K5_K)) continue;
            }
#pragma clang loop unroll(disable)
            for (int64_t i = r + kk; i < r + K5_K; i += 4) {
                const bool have = i < a.rows;
                const k5_floatx4 v = *reinterpret_cast<const k5_floatx4 *>(S + min(i, a.rows - 1) * a.MN);
                const float cl = have ? C[min(i, a.rows - 1) * a.ldC] : 0.f;
#pragma unroll
                for (int x = 0; x < 4; ++x) sum[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(cl, have ? v[x] : 0.f, sum[x], 0, 0, 0);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<k5_floatx4 *>(P + (int64_t)q * a.MN) = k5_floatx4{sum[0][q], sum[1][q], sum[2][q], sum[3][q]};
    }
}

template <int LT>   // L = 16 LT, an even number of tiles
__global__ void __launch_bounds__(NT, 2) mode0_reduce_split_kernel(K5Args a, const uint4 *__restrict__ C3, int64_t groups, const uint32_t *__restrict__ marks)
{
    constexpr bool APART = LT <= 4;   // a step's products are added up before they are added to the sum
    // The instruction's own sums are cut off, not rounded, and always to the same side, which adds up over the steps.  So S is taken with the other
    // sign every TURN steps, and the sum turned with it (64 x 32 x 32, 99,000 slices, one in three stored: 3.9e-7 without, 1.7e-7 so; fp32 2.1e-7).
    constexpr int TURN = APART ? 1 : 4;
    const int tid = threadIdx.x;
    const int wave = tid / 64, lane = tid % 64, kk = lane / 16, col = lane % 16;
    const int c = ((int)blockIdx.y * ((int)blockDim.x / 64) + wave) * 64 + 4 * col;
    const int64_t r0 = (int64_t)blockIdx.x * a.chunk, r1 = min(r0 + a.chunk, a.rows);   // chunks are whole steps
    const float *S = static_cast<const float *>(a.S) + c;
    const uint4 *Cl = C3 + kk * a.L + col;   // part p, step of slices [r, r + 32), l = 16 lt + col: Cl[p * groups * L + r / 8 * L + 16 * lt]
    const int64_t part = groups * a.L;
    k5_floatx4 acc[LT][4];
#pragma unroll
    for (int lt = 0; lt < LT; ++lt)
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[lt][x] = k5_floatx4{0.f, 0.f, 0.f, 0.f};
    k5_floatx4 raw[8];
    auto load_s = [&](int64_t r) {
#pragma unroll
        for (int j = 0; j < 8; ++j) raw[j] = *reinterpret_cast<const k5_floatx4 *>(S + min(r + 8 * kk + j, a.rows - 1) * a.MN);
    };
    uint4 cv[2][3];
    auto load_c = [&](uint4 (&v)[3], int64_t r, int lt) {
#pragma unroll
        for (int p = 0; p < 3; ++p) v[p] = Cl[p * part + r / 8 * a.L + 16 * lt];
    };
    bool left = false;   // some steps are left for fp32
    load_s(r0);
    load_c(cv[0], r0, 0);
    float sign = 1.f;
    int to_turn = TURN;
    for (int64_t r = r0; r < r1; r += K5_K) {
        const int64_t rn = min(r + K5_K, r1 - 1) / K5_K * K5_K;   // the next step, or this one again
        const bool skip = k5_leave<LT>(raw, marks, r / K5_K);
        left |= skip;
        const float scale = skip ? 0.f : sign;
        uint4 s[4][3];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = r + 8 * kk + j < a.rows ? scale * raw[j][x] : 0.f;   // (slices past the last: zero times zero)
            k5_parts(v, s[x]);
        }
        load_s(rn);
#pragma unroll
        for (int lt = 0; lt < LT; ++lt) {
            if (lt + 1 < LT) load_c(cv[(lt + 1) % 2], r, lt + 1);
            else load_c(cv[0], rn, 0);
            __builtin_amdgcn_sched_barrier(0);   // the compiler would otherwise sink these reads below the products
            k5_floatx4 sum[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) sum[x] = APART ? k5_floatx4{0.f, 0.f, 0.f, 0.f} : acc[lt][x];
            auto add = [&](int pc, int ps) {
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    sum[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(k5_bf16, cv[lt % 2][pc]), __builtin_bit_cast(k5_bf16, s[x][ps]), sum[x], 0, 0, 0);
            };
            add(2, 0);
            add(0, 2);
            add(1, 1);
            add(1, 0);
            add(0, 1);
            add(0, 0);
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[lt][x] = APART ? acc[lt][x] + sign * sum[x] : sum[x];
        }
        if (--to_turn == 0 && (APART || r + K5_K < r1)) {
            to_turn = TURN;
            sign = -sign;
            if (!APART)
#pragma unroll
                for (int lt = 0; lt < LT; ++lt)
#pragma unroll
                    for (int x = 0; x < 4; ++x) acc[lt][x] = -acc[lt][x];
        }
    }
    if (!APART)
#pragma unroll
        for (int lt = 0; lt < LT; ++lt)
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[lt][x] *= sign;
    k5_floatx4 none = {0.f, 0.f, 0.f, 0.f};   // ... if every sum is finite
#pragma unroll
    for (int lt = 0; lt < LT; ++lt)
#pragma unroll
        for (int x = 0; x < 4; ++x) none += acc[lt][x] * 0.f;
    const bool again = __any(!(none[0] + none[1] + none[2] + none[3] == 0.f));
    // acc[lt][x][q] = partial(l = 16 lt + 4 kk + q, column c + x)
    float *P = static_cast<float *>(a.partials) + (int64_t)blockIdx.x * a.L * a.MN + c;
#pragma unroll
    for (int lt = 0; lt < LT; ++lt)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<k5_floatx4 *>(P + (int64_t)(16 * lt + 4 * kk + q) * a.MN) = k5_floatx4{acc[lt][0][q], acc[lt][1][q], acc[lt][2][q], acc[lt][3][q]};
    if (!left && !again) return;
    int ln = lane;
    __asm__ volatile("" : "+v"(ln));   // addresses are worked out here: kept over the loop above they cost registers, as `acc` would over this one
    k5_again<LT>(a, r0, r1, ((int)blockIdx.y * ((int)blockDim.x / 64) + wave) * 64 + 4 * (ln % 16), ln / 16, ln % 16, marks, again);
}

// partial(b, l, (m,n)) = sum_{fibers f in chunk b} C(i_f,l) * D(j_f,m) * t(f,n); thread = (m,n)
template <typename T>
__global__ void __launch_bounds__(NT) fiber_reduce_kernel(K5Args a)
{
    __shared__ int s_first;
    const int tid = threadIdx.x;
    const int c = blockIdx.y * NT + tid;
    const int l0 = blockIdx.z * KB_L;
    const int nl = min(KB_L, a.L - l0);
    const int64_t f0 = (int64_t)blockIdx.x * a.chunk, f1 = min(f0 + a.chunk, a.rows);
    const T *C = static_cast<const T *>(a.C);
    const T *D = static_cast<const T *>(a.D);
    const T *Tt = static_cast<const T *>(a.S);
    if (tid == 0) {   // slice that holds fiber f0: last s with pos2[s] <= f0
        int lo = 0, hi = a.nslices;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.pos2[mid] <= f0) lo = mid; else hi = mid;
        }
        s_first = lo;
    }
    __syncthreads();
    int s = s_first;
    int64_t s_end = a.pos2[s + 1];
    const int m = c < a.MN ? c / a.N : 0, n = c < a.MN ? c % a.N : 0;
    T acc[KB_L];
#pragma unroll
    for (int l = 0; l < KB_L; ++l) acc[l] = T(0);
    T crow[KB_L];
    auto load_c = [&](int slice) {
        const int64_t i = a.crd1[slice];
#pragma unroll
        for (int l = 0; l < KB_L; ++l) crow[l] = l < nl ? C[i * a.ldC + l0 + l] : T(0);
    };
    load_c(s);
    for (int64_t f = f0; f < f1; ++f) {
        if (f >= s_end) {   // uniform: every thread walks the same fibers
            ++s;
            s_end = a.pos2[s + 1];
            load_c(s);
        }
        const int64_t j = a.crd2[f];
        const T dt = D[j * a.ldD + m] * Tt[f * a.N + n];
#pragma unroll
        for (int l = 0; l < KB_L; ++l) acc[l] += crow[l] * dt;
    }
    if (c < a.MN) {
        T *P = static_cast<T *>(a.partials) + (int64_t)blockIdx.x * a.L * a.MN;
        for (int l = 0; l < nl; ++l) P[(int64_t)(l0 + l) * a.MN + c] = acc[l];
    }
}

// LINEAR: the perfectly nested loop of Figure 2a, nothing factored out: every stored entry is multiplied with one
// element of each of the three factors for every (l, m, n).  A workgroup walks a contiguous chunk of fibers; a
// thread owns KB_L output elements e = (l, m, n) of one block of KB_L * NT elements (blockIdx.y) and keeps their
// sums in registers; the partial tiles of the chunks are added by sum_partials like those of the other schedules.
template <typename T>
__global__ void __launch_bounds__(NT) linear_all_kernel(K5Args a, const int32_t *__restrict__ pos3, const int32_t *__restrict__ crd3,
                                                        const T *__restrict__ vals, const T *__restrict__ E, int64_t ldE)
{
    __shared__ int s_first;
    const int tid = threadIdx.x;
    const int64_t elems = (int64_t)a.L * a.MN;
    const int64_t f0 = (int64_t)blockIdx.x * a.chunk, f1 = min(f0 + a.chunk, a.rows);
    const T *C = static_cast<const T *>(a.C);
    const T *D = static_cast<const T *>(a.D);
    if (tid == 0) {   // slice that holds fiber f0: last s with pos2[s] <= f0
        int lo = 0, hi = a.nslices;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.pos2[mid] <= f0) lo = mid; else hi = mid;
        }
        s_first = lo;
    }
    __syncthreads();
    int l[KB_L], m[KB_L], n[KB_L];
    bool ok[KB_L];
    T acc[KB_L];
#pragma unroll
    for (int r = 0; r < KB_L; ++r) {
        const int64_t e = ((int64_t)blockIdx.y * KB_L + r) * NT + tid;
        ok[r] = e < elems;
        const int64_t ec = ok[r] ? e : 0;
        l[r] = (int)(ec / a.MN);
        m[r] = (int)((ec % a.MN) / a.N);
        n[r] = (int)(ec % a.N);
        acc[r] = T(0);
    }
    int s = s_first;
    int64_t s_end = a.pos2[s + 1];
    int64_t i = a.crd1[s];
    for (int64_t f = f0; f < f1; ++f) {
        if (f >= s_end) {   // uniform: every thread walks the same fibers
            ++s;
            s_end = a.pos2[s + 1];
            i = a.crd1[s];
        }
        const int64_t j = a.crd2[f];
        for (int z = pos3[f]; z < pos3[f + 1]; ++z) {
            const int64_t k = crd3[z];
            const T v = vals[z];
#pragma unroll
            for (int r = 0; r < KB_L; ++r) acc[r] += v * C[i * a.ldC + l[r]] * D[j * a.ldD + m[r]] * E[k * ldE + n[r]];
        }
    }
    T *P = static_cast<T *>(a.partials) + (int64_t)blockIdx.x * elems;
#pragma unroll
    for (int r = 0; r < KB_L; ++r)
        if (ok[r]) P[((int64_t)blockIdx.y * KB_L + r) * NT + tid] = acc[r];
}

// A(e) = sum over chunks b of partial(b, e), in an order fixed by the launch: a workgroup owns EW output
// elements, its NT / EW groups of lanes take the chunks round robin and their sums are added in group order.
// Every output element is written.  Small outputs over many chunks (16^3: 4096 elements, 507 chunks) leave 64-element
// workgroups a chain of 127 reads each and the chip mostly idle; 16 elements keep the reads whole 64-byte segments, four
// times the workgroups and a quarter of the chain (11 -> 5.5 us).
template <typename T, int EW>
__global__ void __launch_bounds__(NT) sum_partials_kernel(const T *__restrict__ partials, int nchunks, int64_t elems, T *__restrict__ out)
{
    __shared__ T part_s[NT];
    const int lane = threadIdx.x % EW, part = threadIdx.x / EW;
    const int64_t e = (int64_t)blockIdx.x * EW + lane;
    T s = T(0);
    if (e < elems) {
#pragma unroll 8
        for (int b = part; b < nchunks; b += NT / EW) s += partials[(int64_t)b * elems + e];
    }
    part_s[threadIdx.x] = s;
    __syncthreads();
    if (part == 0 && e < elems) {
        T tot = part_s[lane];
        for (int w = 1; w < NT / EW; ++w) tot += part_s[w * EW + lane];
        out[e] = tot;
    }
}

template <typename T>
sc_status run_ttmc_all(const sc_plan *p, const sc_csf_view *sp, const sc_dense_view *fac, void *out, void *ws, hipStream_t stream)
{
    const sc_plan *in = p->inner;
    const sc_dense_view inner_fac[2] = {fac[1], fac[2]};
    char *wsb = static_cast<char *>(ws);
    const int L = (int)p->fcols[0], M = (int)p->fcols[1], N = (int)p->fcols[2], MN = M * N;
    const int64_t elems = (int64_t)L * MN;
    Launcher ln{p, stream};
    K5Args a = {};
    a.C = fac[0].data; a.ldC = fac[0].ld;
    a.D = fac[1].data; a.ldD = fac[1].ld;
    a.L = L; a.M = M; a.N = N; a.MN = MN;
    a.partials = wsb + p->k5_partials_offset;
    a.chunk = (int32_t)p->k5_chunk;
    const dim3 grid((unsigned)p->k5_nchunks, (unsigned)((MN + NT - 1) / NT), (unsigned)((L + KB_L - 1) / KB_L));
    if (p->nnz == 0) {   // nothing stored: the output is zero
        launch_fill<T>(ln, static_cast<T *>(out), elems, "fill_output");
        return ln.status;
    }
    if (p->k5_variant == 0) {
        // the unfactored nest over all stored entries
        a.crd1 = sp->crd[0]; a.pos2 = sp->pos[1]; a.crd2 = sp->crd[1];
        a.rows = p->nfib[1];
        a.nslices = (int32_t)p->nfib[0];
        const dim3 lgrid((unsigned)p->k5_nchunks, (unsigned)((elems + (int64_t)KB_L * NT - 1) / ((int64_t)KB_L * NT)), 1);
        ln.begin("ttmc_all_linear_nest");
        linear_all_kernel<T><<<lgrid, NT, 0, stream>>>(a, sp->pos[2], sp->crd[2], static_cast<const T *>(sp->vals),
                                                       static_cast<const T *>(fac[2].data), fac[2].ld);
        ln.end();
    } else if (p->k5_variant == 1) {
        // t(f,:) per fiber by the leaf traversal of the inner plan (its first FISSIONED kernel), then the fiber reduction
        Launcher li{in, stream};
        void *T1 = wsb + p->k5_inner_ws_offset + in->inter[0].offset;
        void *partials_a = in->deterministic ? wsb + p->k5_inner_ws_offset + in->det_a.slot_offset : nullptr;
        sc_status st = launch_leaf_producer(in, li, sp->vals, fac[2], T1, N, "ttmc_all_traverse", partials_a);
        if (st != SC_OK) return st;
        st = launch_fixup(in, li, in->det_a, wsb + p->k5_inner_ws_offset, T1);
        if (st != SC_OK) return st;
        a.S = T1;
        a.crd1 = sp->crd[0]; a.pos2 = sp->pos[1]; a.crd2 = sp->crd[1];
        a.rows = p->nfib[1];
        a.nslices = (int32_t)p->nfib[0];
        ln.begin("ttmc_all_fiber_reduce");
        fiber_reduce_kernel<T><<<grid, NT, 0, stream>>>(a);
        ln.end();
    } else {
        void *S = wsb + p->k5_s_offset;
        const sc_status st = launch_plan(in, sp, inner_fac, S, wsb + p->k5_inner_ws_offset, stream);
        if (st != SC_OK) return st;
        a.S = S;
        a.rows = p->dims[0];
        if (p->k5_mfma_reduce) {
            if constexpr (sizeof(T) == 4) {
                if (MN % 64 != 0) return SC_ERR_SCHED_UNSUPPORTED;
                if (p->k5_split_offset != SIZE_MAX) {
                    const int64_t groups = (a.rows + K5_K - 1) / K5_K * (K5_K / 8);
                    uint4 *C3 = reinterpret_cast<uint4 *>(wsb + p->k5_split_offset);
                    ln.begin("ttmc_all_split");
                    uint32_t *marks = reinterpret_cast<uint32_t *>(C3 + 3 * groups * L);
                    k5_split_kernel<<<(unsigned)(groups * L / NT), NT, 0, stream>>>(static_cast<const float *>(a.C), a.ldC, a.rows, L, groups, C3, marks);
                    ln.end();
                    const int strips = MN / 64, waves = strips % 4 == 0 ? 4 : strips % 2 == 0 ? 2 : 1;   // wavefronts per workgroup
                    const dim3 sgrid((unsigned)p->k5_nchunks, (unsigned)(strips / waves), 1);
                    ln.begin("ttmc_all_mode0_reduce_split");
                    auto reduce = [&](auto lt) { mode0_reduce_split_kernel<decltype(lt)::value><<<sgrid, 64 * waves, 0, stream>>>(a, C3, groups, marks); };
                    if (L == 64) reduce(std::integral_constant<int, 4>{});
                    else if (L == 128) reduce(std::integral_constant<int, 8>{});
                    else return SC_ERR_SCHED_UNSUPPORTED;
                    ln.end();
                } else {
                // 64 columns per wavefront, 16 up to two wavefronts of 64 per compute unit.  Whole calls at 512 wavefronts of 64: 128 x 32 x
                // 32 42.2 us with 64 columns, 38.2 with 16; at 628: 44.6 and 42.5 at 128 x 16 x 16, but 32.2 and 33.6 at 32 x 16 x 16; at
                // 1008 64 columns are equal or ahead at every L (64 x 32 x 32: 36.9 and 38.3).
                const bool narrow = p->k5_nchunks * (MN / 64) <= (int64_t)2 * p->n_cu;
                const int cols = narrow ? 16 : 64, strips = (int)(MN / cols);
                const int waves = strips % 4 == 0 ? 4 : strips % 2 == 0 ? 2 : 1;   // wavefronts per workgroup
                const dim3 mgrid((unsigned)p->k5_nchunks, (unsigned)(strips / waves), 1);
                auto reduce = [&](auto lt) {
                    constexpr int LT = decltype(lt)::value;
                    if (narrow) mode0_reduce_mfma_kernel<LT, 1><<<mgrid, 64 * waves, 0, stream>>>(a);
                    else mode0_reduce_mfma_kernel<LT, 4><<<mgrid, 64 * waves, 0, stream>>>(a);
                };
                ln.begin("ttmc_all_mode0_reduce_mfma");
                if (L == 16) reduce(std::integral_constant<int, 1>{});
                else if (L == 32) reduce(std::integral_constant<int, 2>{});
                else if (L == 64) reduce(std::integral_constant<int, 4>{});
                else if (L == 128) reduce(std::integral_constant<int, 8>{});
                else return SC_ERR_SCHED_UNSUPPORTED;
                ln.end();
                }
            } else {
                return SC_ERR_SCHED_UNSUPPORTED;
            }
        } else {
            ln.begin("ttmc_all_mode0_reduce");
            mode0_reduce_kernel<T><<<grid, NT, 0, stream>>>(a);
            ln.end();
        }
    }
    ln.begin("ttmc_all_sum_partials");
    // 16 elements per workgroup while 64 would leave compute units without one and there are chunks to share out
    if (elems <= (int64_t)64 * p->n_cu && p->k5_nchunks >= 64)
        sum_partials_kernel<T, 16><<<(unsigned)((elems + 15) / 16), NT, 0, stream>>>(static_cast<const T *>(a.partials), (int)p->k5_nchunks,
                                                                                     elems, static_cast<T *>(out));
    else
        sum_partials_kernel<T, 64><<<(unsigned)((elems + 63) / 64), NT, 0, stream>>>(static_cast<const T *>(a.partials), (int)p->k5_nchunks,
                                                                                     elems, static_cast<T *>(out));
    ln.end();
    return ln.status;
}

}  // namespace

sc_status launch_ttmc_all(const sc_plan *p, const sc_csf_view *sp, const sc_dense_view *fac, void *out, void *ws, hipStream_t stream)
{
    if (!p->inner) return SC_ERR_SCHED_UNSUPPORTED;
    return p->dtype == SC_F64 ? run_ttmc_all<double>(p, sp, fac, out, ws, stream) : run_ttmc_all<float>(p, sp, fac, out, ws, stream);
}

}  // namespace sck
