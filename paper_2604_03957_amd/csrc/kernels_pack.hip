// Ternarise + bit-pack activations, sign-pack weights (paper: "Ternary Function" and sign
// equations; "Instruction-level Parallel Bitpack").  Bandwidth-bound streaming kernels: every
// lane takes 8 consecutive elements with one 128-bit (fp16) or 64-bit (int8) load, turns them
// into one byte per plane, and the four lanes of a quad assemble a 32-bit plane word.
#include "bwta_internal.h"

namespace bwta {

namespace {

constexpr int kThreads = 256;
// four groups per thread only when that still leaves a few workgroups per compute unit
constexpr int64_t kQuadGroupMinThreads = 1024 * kThreads;

// OR a per-lane byte into its quad's 32-bit word (lane q of the quad supplies byte q).
__device__ __forceinline__ uint32_t quad_word(uint32_t byte, int lane)
{
    uint32_t v = byte << (8 * (lane & 3));
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, true);  // quad_perm [2,3,0,1]
    return v;
}

// One group of 8 elements per thread: small launches, rows of fewer than 8 elements, int8 input.
template <int DTYPE>  // 0 = fp16 -> ternary, 1 = int8 ternary, 2 = fp16 -> boolean (the bool function: 1 iff a >= 0.5 s)
__global__ __launch_bounds__(kThreads) void k_quantize_pack(const void *__restrict__ A, int64_t lda,
                                                            ScaleArg s_a, int M, int K, int rw,
                                                            uint32_t *__restrict__ mask,
                                                            uint32_t *__restrict__ sign)
{
    const int c8 = rw * 4;  // byte-groups (8 elements) per packed row, a multiple of 16
    const int64_t total = (int64_t)M * c8;
    const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (gid >= total) return;  // whole quads leave together (total % 4 == 0)
    const int m = (int)(gid / c8);
    const int c = (int)(gid - (int64_t)m * c8);
    const int k0 = c * 8;
    uint32_t nz = 0, neg = 0;
    if (DTYPE == 0 || DTYPE == 2) {
        // the scale is requested before the data and by every lane (without a scale: a dropped read
        // of the first element), so the two requests share one memory round trip
        const bool have_scale = s_a.mode != 0 && s_a.ptr != nullptr;
        const uint16_t s_bits = *(have_scale ? s_a.ptr + (s_a.mode == 1 ? 0 : m) : (const uint16_t *)A);
        const uint16_t *row = (const uint16_t *)A + (int64_t)m * lda;
        const uint4 x = K >= 8 ? finish_group(request_group(row, k0, K), k0, K) : short_row_group(row, k0, K);
        ternary_flags<DTYPE == 2>(x, ternary_thresholds(have_scale ? s_bits : 0x3c00u, true), nz, neg);
    } else {
        const int8_t *row = (const int8_t *)A + (int64_t)m * lda;
        unsigned long long v = 0;
        if (K >= 8) {  // as request_group / finish_group
            __builtin_memcpy(&v, row + (k0 <= K - 8 ? k0 : K - 8), 8);
            const int drop = k0 + 8 - K;
            if (drop > 0) v = drop >= 8 ? 0 : v >> (8 * drop);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (k0 == 0 && i < K) v |= (unsigned long long)(uint8_t)row[i] << (8 * i);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int8_t e = (int8_t)(v >> (8 * i));
            nz |= (uint32_t)(e != 0) << i;
            neg |= (uint32_t)(e < 0) << i;
        }
    }
    const int lane = threadIdx.x & 63;
    uint32_t wm = quad_word(nz, lane);
    uint32_t ws = quad_word(neg, lane);
    const int64_t widx = (int64_t)m * rw + (c >> 2);
    if ((lane & 3) == 0) mask[widx] = wm;
    if (DTYPE != 2 && (lane & 3) == 1) sign[widx] = ws;
}

// The same operation for fp16 rows of at least 8 elements (any alignment): a thread takes four groups of
// one row, a quarter row apart, and issues its scale request and all four 128-bit loads before anything is
// used, so four times the bytes are in flight per wavefront.  Index space: row m, word w0 in the first
// quarter of the row, quad lane q; group u is byte-group 4 (w0 + u rw / 4) + q.
// Bound: HBM.  The thresholds are compared in packed half precision (ternary_flags: 1.5 instructions per
// element for the bool function, 3 for the ternary one; converting and comparing in fp32 took 7 and kept
// the vector ALU busy for as long as the memory): 65536 rows of 2048 (268 MB) 40 us = 6.7 TB/s either way,
// 8192 rows (34 MB, in the L2) 4.7 us.  Workgroups take the rows in order: from the last to the first, to
// meet in the memory-side cache what a scale pass just left there, loses the L2 of the own XCD and gains
// nothing beyond it (scale + boolean pack of 34 MB: 14.2 against 10.1 us).
template <int DTYPE>  // 0 = ternary, 2 = boolean
__global__ __launch_bounds__(kThreads) void k_quantize_pack_vec(const uint16_t *__restrict__ A, int64_t lda,
                                                                ScaleArg s_a, int M, int K, int rw,
                                                                uint32_t *__restrict__ mask,
                                                                uint32_t *__restrict__ sign)
{
    const int64_t total = (int64_t)M * rw;  // threads with work: M rows x rw / 4 words x 4 lanes
    const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool live = gid < total;  // whole quads together (rw % 4 == 0)
    const int64_t gc = live ? gid : 0;
    const int m = (int)(gc / rw), rem = (int)(gc - (int64_t)m * rw);
    const int w0 = rem >> 2, q = rem & 3, qw = rw >> 2;
    const bool have_scale = s_a.mode != 0 && s_a.ptr != nullptr;
    const uint16_t s_bits = *(have_scale ? s_a.ptr + (s_a.mode == 1 ? 0 : m) : A);
    const uint16_t *row = A + (int64_t)m * lda;
    uint4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = request_group(row, 8 * (4 * (w0 + u * qw) + q), K);
    __builtin_amdgcn_sched_barrier(0);
    const TernaryThr thr = ternary_thresholds(have_scale ? s_bits : 0x3c00u, true);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int w = w0 + u * qw;
        uint32_t nz, neg;
        ternary_flags<DTYPE == 2>(finish_group(x[u], 8 * (4 * w + q), K), thr, nz, neg);
        const uint32_t wm = quad_word(nz, lane);
        const uint32_t ws = DTYPE == 2 ? 0u : quad_word(neg, lane);
        const int64_t widx = (int64_t)m * rw + w;
        if (live && q == 0) mask[widx] = wm;
        if (DTYPE != 2 && live && q == 1) sign[widx] = ws;
    }
}

template <int DTYPE>
__global__ __launch_bounds__(kThreads) void k_pack_weights(const void *__restrict__ W, int64_t ldw,
                                                           int N, int K, int rw,
                                                           uint32_t *__restrict__ wsign, int vec_ok)
{
    const int c8 = rw * 4;
    const int64_t total = (int64_t)N * c8;
    const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (gid >= total) return;
    const int n = (int)(gid / c8);
    const int c = (int)(gid - (int64_t)n * c8);
    const int k0 = c * 8;
    const int nvalid = K - k0 >= 8 ? 8 : (K - k0 > 0 ? K - k0 : 0);
    uint32_t bits = 0;
    if (DTYPE == 0) {
        const uint16_t *row = (const uint16_t *)W + (int64_t)n * ldw;
        uint16_t v[8];
        if (nvalid == 8 && vec_ok) {
            uint4 q = *(const uint4 *)(row + k0);
            v[0] = q.x & 0xffff; v[1] = q.x >> 16; v[2] = q.y & 0xffff; v[3] = q.y >> 16;
            v[4] = q.z & 0xffff; v[5] = q.z >> 16; v[6] = q.w & 0xffff; v[7] = q.w >> 16;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = i < nvalid ? row[k0 + i] : (uint16_t)0;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float w = half_bits_to_float(v[i]);
            bits |= (uint32_t)((i < nvalid) && !(w >= 0.0f)) << i;  // "otherwise" includes NaN
        }
    } else {
        const int8_t *row = (const int8_t *)W + (int64_t)n * ldw;
        if (nvalid == 8 && vec_ok) {
            uint2 q = *(const uint2 *)(row + k0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                bits |= ((q.x >> (8 * i + 7)) & 1u) << i;
                bits |= ((q.y >> (8 * i + 7)) & 1u) << (4 + i);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                int8_t w = i < nvalid ? row[k0 + i] : (int8_t)0;
                bits |= (uint32_t)(w < 0) << i;
            }
        }
    }
    const int lane = threadIdx.x & 63;
    uint32_t word = quad_word(bits, lane);
    if ((lane & 3) == 0) wsign[(int64_t)n * rw + (c >> 2)] = word;
}

// nnz[m] = popcount of mask row m; one wavefront per row.
__global__ __launch_bounds__(kThreads) void k_row_popcount(const uint32_t *__restrict__ mask, int M,
                                                           int rw, int32_t *__restrict__ nnz)
{
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (m >= M) return;
    int c = 0;
    for (int w = lane; w < rw; w += 64) c += __popc(mask[(int64_t)m * rw + w]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if (lane == 0) nnz[m] = c;
}

// ---- weight preparation from full-precision weights, and the activation scale's starting value ----
//
// Binary16 values are integers in units of 2^-24 (|v| < 2^40), so a row's sum is an exact 64-bit
// integer whatever the order of the additions, and "W[n,k] - mean >= 0" is the integer test
// K * W[n,k] >= sum.  Every discrete decision is therefore identical to exact arithmetic.

// non-negative double -> binary16 bits, round to nearest even, straight from the 53-bit significand
// (going through fp32 would round twice)
__device__ __forceinline__ uint16_t double_to_half_bits(double x)
{
    if (!(x > 0.0)) return 0;
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    int e = (int)((b >> 52) & 0x7ff) - 1023;
    if (e > 15) return 0x7c00;
    if (e < -26) return 0;  // below half of the smallest subnormal
    const unsigned long long mant = (b & ((1ull << 52) - 1)) | (1ull << 52);
    const int shift = 42 + (e < -14 ? -14 - e : 0);  // bits dropped: keep 11 (normal) or fewer (subnormal)
    unsigned long long q = mant >> shift;
    const unsigned long long rem = mant & ((1ull << shift) - 1), half = 1ull << (shift - 1);
    if (rem > half || (rem == half && (q & 1))) ++q;
    if (e < -14) return (uint16_t)q;  // subnormal, or exactly the smallest normal (q = 1024)
    if (q == 2048) {
        q = 1024;
        ++e;
    }
    if (e > 15) return 0x7c00;
    return (uint16_t)(((e + 15) << 10) | (int)(q - 1024));
}

__device__ __forceinline__ uint16_t half_of(const uint4 &q, int i)
{
    const uint32_t w = i < 2 ? q.x : (i < 4 ? q.y : (i < 6 ? q.z : q.w));
    return (uint16_t)(w >> (16 * (i & 1)));
}

// A per-thread sum of at most 128 finite binary16 values is a multiple of 2^-24 below 2^23: exact
// in a double whatever the order.  This turns it into the integer count of 2^-24.
__device__ __forceinline__ long long double_units(double s) { return (long long)(s * 16777216.0); }

// The smallest value on the binary16 grid that is >= c * 2^-24 (c an integer count of 2^-24), as a
// float; +Inf if there is none.  For every finite binary16 x with integer count X:
// X >= c  <=>  float(x) >= result, so a 64-bit comparison per element becomes one float compare.
__device__ __forceinline__ float half_grid_ceil(long long c)
{
    const long long top = 65504ll << 24;
    if (c > top) return __builtin_inff();
    const bool negative = c < 0;
    unsigned long long a = (unsigned long long)(negative ? -c : c);
    if (a > (unsigned long long)top) a = (unsigned long long)top;  // only for c < -top: every finite x is >= c
    const int p = 63 - __builtin_clzll(a | 1ull);                   // position of the leading one
    if (p > 10) {  // grid spacing 2^(p-10): magnitudes round down for a negative bound, up for a positive one
        const unsigned long long sp = 1ull << (p - 10);
        a = negative ? (a & ~(sp - 1)) : ((a + sp - 1) & ~(sp - 1));
    }
    const float v = (float)(long long)a * 5.9604644775390625e-08f;  // at most 12 significant bits: exact
    return negative ? -v : v;
}

// ---- exact sums of binary16 magnitudes ----------------------------------------------------------
//
// The 15 magnitude bits of a binary16 value, put at the same place of a double (exponent field on
// exponent field), are that value times 2^-1008: exactly, subnormals included, because a double whose
// exponent field is 0 is scaled by the same rule.  So a magnitude becomes a double with one shift and
// one mask and joins the sum with one addition, three full-rate instructions, where a conversion
// through float, the exclusion of non-finite values and a second conversion took seven.  Per-thread
// sums are exact (at most 128 values, see double_units) with binary64 subnormals on, the HIP default.
// Non-finite values are noticed from the sum of squares, one dot-product instruction per two
// values; a thread that holds one adds its values again with the exclusion.
__device__ __forceinline__ float add_squares(uint32_t two, float sum)
{
    typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
    half2_t h;
    __builtin_memcpy(&h, &two, 4);
    return __builtin_amdgcn_fdot2(h, h, sum, false);
}

// false for Inf and for NaN; on the bits, because the compiler takes the dot product to be never NaN
__device__ __forceinline__ bool is_finite_sum(float squares) { return (__float_as_uint(squares) & 0x7f800000u) != 0x7f800000u; }

struct MagnitudeSum {
    double even = 0.0, odd = 0.0;
    float squares = 0.0f;

    __device__ __forceinline__ void add(const uint4 &x)
    {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            even += __hiloint2double((int)((w[i] << 10) & 0x01fffc00u), 0);
            odd += __hiloint2double((int)((w[i] >> 6) & 0x01fffc00u), 0);
            squares = add_squares(w[i], squares);
        }
    }
    __device__ __forceinline__ bool all_finite() const { return is_finite_sum(squares); }
    __device__ __forceinline__ long long units() const { return (long long)ldexp(even + odd, 1008 + 24); }
};

// the same count of 2^-24 with NaN and Inf left out
template <int NG>
__device__ __forceinline__ long long finite_magnitude_units(const uint4 (&x)[NG])
{
    double part = 0.0;
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint16_t h = half_of(x[g], i) & 0x7fff;
            part += (double)(h < 0x7c00 ? half_bits_to_float(h) : 0.0f);
        }
    return double_units(part);
}

template <int NG>
__device__ __forceinline__ long long magnitude_units(const uint4 (&x)[NG])
{
    MagnitudeSum sum;
#pragma unroll
    for (int g = 0; g < NG; ++g) sum.add(x[g]);
    return sum.all_finite() ? sum.units() : finite_magnitude_units(x);
}

// groups first, first + step, ..: all requested before any is used; the row's end is only looked at by
// waves of a launch whose last groups reach it (step groups go with one pass over the row)
template <int NG>
__device__ __forceinline__ void load_row(const uint16_t *row, int first, int step, int K, uint4 (&x)[NG])
{
    if (K >= 8) {
#pragma unroll
        for (int g = 0; g < NG; ++g) x[g] = request_group(row, 8 * (first + step * g), K);
        __builtin_amdgcn_sched_barrier(0);
        if (8 * step * NG > K) {
#pragma unroll
            for (int g = 0; g < NG; ++g) x[g] = finish_group(x[g], 8 * (first + step * g), K);
        }
    } else {
#pragma unroll
        for (int g = 0; g < NG; ++g) x[g] = short_row_group(row, 8 * (first + step * g), K);
    }
}

// sum over L consecutive lanes (4 <= L <= 64); every lane gets it
template <int CTRL>
__device__ __forceinline__ int dpp_move(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}

template <int CTRL>
__device__ __forceinline__ long long dpp_move(long long x)
{
    return (long long)((unsigned long long)(uint32_t)dpp_move<CTRL>((int)(x >> 32)) << 32 |
                       (uint32_t)dpp_move<CTRL>((int)x));
}

template <int L, typename T>
__device__ __forceinline__ T lane_group_sum(T v)
{
    v += dpp_move<0xb1>(v);                 // quad_perm [1,0,3,2]
    v += dpp_move<0x4e>(v);                 // quad_perm [2,3,0,1]
    if (L >= 8) v += dpp_move<0x141>(v);    // row_half_mirror: lane i <-> 7 - i
    if (L >= 16) v += dpp_move<0x140>(v);   // row_mirror: i <-> 15 - i
    if (L >= 32) v += __shfl_xor(v, 16);
    if (L >= 64) v += __shfl_xor(v, 32);
    return v;
}

// fp16(2 S / (K 2^24)) of a row whose magnitudes sum to S units of 2^-24
__device__ __forceinline__ uint16_t scale_bits(long long S, int K)
{
    return double_to_half_bits((double)S / ((double)K * 8388608.0));
}

// s[m] = 2 * mean_k |A[m, k]| (exact integer sum, one division, one rounding).  Bound: HBM, one read of
// A.  Rows up to 4096 elements: L lanes of one wavefront per row, NG groups of 8 elements per lane, no
// barrier and no LDS; a wavefront takes R sets of 64 / L rows so that short rows still keep R NG loads
// per lane in flight and share the reduction's and the division's fixed cost (each of the first R lanes
// of a row's group finishes one of the R rows).  Measured on an attention block's operands against
// one workgroup of 256 threads per row (whose barriers, 64-bit shuffles and division a row of 128 or 2048
// elements cannot pay for): 65536 rows of 128: 61 -> 5.9 us; 65536 rows of 2048 (268 MB): 67 -> 39.5 us =
// 6.8 TB/s.
template <int L, int NG, int R>
__global__ __launch_bounds__(kThreads) void k_act_scale_wave(const uint16_t *__restrict__ A, int64_t lda, int M, int K,
                                                             uint16_t *__restrict__ s)
{
    constexpr int RPW = 64 / L;  // rows side by side in a wavefront
    static_assert(R <= L, "one lane of a row's group per set");
    const int lane = threadIdx.x & 63, cl = lane % L;
    const int64_t row0 = ((int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)) * (R * RPW) + lane / L;
    uint4 x[R][NG];
    auto row_of = [&](int r) { return A + (row0 + r * RPW < M ? row0 + r * RPW : M - 1) * lda; };
    if (K >= 8) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int g = 0; g < NG; ++g) x[r][g] = request_group(row_of(r), 8 * (cl + L * g), K);
        __builtin_amdgcn_sched_barrier(0);
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int g = 0; g < NG; ++g) x[r][g] = short_row_group(row_of(r), 8 * (cl + L * g), K);
    }
    long long mine = 0;  // lane r of the group keeps the sum of set r
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (K >= 8 && 8 * L * NG > K) {
#pragma unroll
            for (int g = 0; g < NG; ++g) x[r][g] = finish_group(x[r][g], 8 * (cl + L * g), K);
        }
        const long long S = lane_group_sum<L>(magnitude_units(x[r]));
        mine = cl == r ? S : mine;
    }
    const int64_t m = row0 + cl * RPW;
    if (cl < R && m < M) s[m] = scale_bits(mine, K);
}

// Longer rows, and rows of more than 512 elements where there are few of them, so that a row's latency counts and not
// the bytes: one workgroup of NT threads per row.  16 rows of 3000: 3.1 -> 2.6 us; 1024: 3.4 either way.
template <int NG, int NT>
__global__ __launch_bounds__(NT) void k_act_scale(const uint16_t *__restrict__ A, int64_t lda, int K,
                                                        uint16_t *__restrict__ s)
{
    __shared__ long long s_ll[NT / 64];
    const int64_t m = blockIdx.x;
    uint4 x[NG];
    load_row<NG>(A + m * lda, threadIdx.x, NT, K, x);
    const long long part = lane_group_sum<64>(magnitude_units(x));
    if ((threadIdx.x & 63) == 0) s_ll[threadIdx.x >> 6] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long S = 0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) S += s_ll[i];
        s[m] = scale_bits(S, K);
    }
}

// One group of NT threads (a wavefront or a workgroup of 256) per output channel: mean (exact),
// sign(W - mean) packed like bwta_pack_weights, s_w = mean |W - mean|.  With X the integer count of 2^-24
// of an element and S the row's exact sum, "W - mean < 0" is X K < S, i.e. X < ceil(S / K): a compare of
// binary16 values against the smallest one that is not below that bound.  The sum of |X K - S| over the
// finite elements equals K (S - 2 Sn) - S (n - 2 nn) with Sn, nn the sum and count of the finite elements
// below the mean and n the count of finite elements, so the second pass needs only exact per-thread
// sums again; the final combination is done in double (one division, one rounding to binary16).
// Bound: HBM.  The row stays in registers between the passes.  Both sums are exact: in fp32 by groups of 8 where
// the values are small enough (SmallSum below: weights, as a rule), else on the double form of a binary16
// value (MagnitudeSum above, here with its sign).  The compare is one packed subtraction whose
// sign survives rounding (ternary_thresholds) and one packed minimum per two elements, and a masked
// element adds zero: about 5 instructions per element in all, 9 with the double form.  Wavefronts that hold a
// NaN or an Inf go through their elements one by one instead.  A row of up to 4096 elements takes one wavefront and
// no barrier.  Measured on fp16 [4096, 11008]: two conversions and three selects per element and pass 48.7 us, the
// double form 24.0, fp32 by groups 21.1 us (4.5 TB/s); with the double form one or two wavefronts per row were
// 4 to 15 % slower there (registers), at K = 4096 one is 20 % ahead of four.  Rows beyond 16384, 16 groups per thread
// (two wavefronts per SIMD) where 1024 threads converted before: [4096, 20000] 141 -> 55 us.
struct SignedSum {
    double even = 0.0, odd = 0.0;

    __device__ __forceinline__ void add(uint32_t two)
    {
        int low;  // the low half's sign-extended bits << 10, in one instruction
        asm("v_mad_i32_i16 %0, %1, %2, 0" : "=v"(low) : "v"(two), "s"(1024));
        even += __hiloint2double(low & (int)0x81fffc00u, 0);
        odd += __hiloint2double((int)two >> 6 & (int)0x81fffc00u, 0);
    }
    __device__ __forceinline__ long long units() const { return (long long)ldexp(even + odd, 1008 + 24); }
};

// The same sum where every group of 8 has squares that add to less than 1/8, at one instruction per element
// instead of three.  By Cauchy-Schwarz any partial sum of a group then lies below sqrt(8 / 8) = 1, so it is less
// than 2^24 units of 2^-24 and exact in fp32; the groups' sums are added as integers.  (Weights of a standard
// deviation up to 0.08 or so pass; any others take the double form.)
struct SmallSum {
    int units = 0;  // at most 16 groups of less than 2^24: below 2^28

    __device__ __forceinline__ void add(const uint32_t (&w)[4])
    {
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel_hi:[1,0,0]" : "+v"(s) : "v"(w[i]));
            asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(s) : "v"(w[i]));
        }
        units += (int)(s * 16777216.0f);
    }
    // squares: the bits of a sum of squares, which Inf and NaN fail; 0.12 leaves room for its rounding
    static __device__ __forceinline__ bool exact_below(uint32_t squares) { return squares < __float_as_uint(0.12f); }
};

// the wavefront's sums; lane 0 of every wavefront leaves them in LDS when a row has several
template <int NT>
__device__ __forceinline__ void wave_sums(long long &a, int &b, long long *scratch /* [2 * NT / 64] */)
{
    a = lane_group_sum<64>(a);
    if (__any(b != 0)) b = lane_group_sum<64>(b);
    if constexpr (NT > 64) {
        if ((threadIdx.x & 63) == 0) {
            scratch[2 * (threadIdx.x >> 6)] = a;
            scratch[2 * (threadIdx.x >> 6) + 1] = b;
        }
    }
}

template <int NT>
__device__ __forceinline__ void row_sums(long long &a, int &b, const long long *scratch)
{
    if constexpr (NT > 64) {
        a = scratch[0], b = (int)scratch[1];
#pragma unroll
        for (int i = 1; i < NT / 64; ++i) a += scratch[2 * i], b += (int)scratch[2 * i + 1];
    }
}

template <int NG, int NT>
__global__ __launch_bounds__(NT) void k_prepare_weights(const uint16_t *__restrict__ W, int64_t ldw, int K, int rw,
                                                        uint32_t *__restrict__ wsign, uint16_t *__restrict__ s_w)
{
    __shared__ long long s_mean[2 * NT / 64], s_below[2 * NT / 64];
    const int64_t n = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const uint16_t *row = W + n * ldw;
    uint4 x[NG];
    load_row<NG>(row, threadIdx.x, NT, K, x);

    uint32_t squares = 0;  // the largest sum of a group's squares, as its bits
    SmallSum small_sum;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const uint32_t w[4] = {x[g].x, x[g].y, x[g].z, x[g].w};
        small_sum.add(w);
        float sq = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) sq = add_squares(w[i], sq);
        squares = max(squares, __float_as_uint(sq));
    }
    const bool small = __all(SmallSum::exact_below(squares));
    long long S = small_sum.units;
    if (!small) {
        SignedSum sum;
#pragma unroll
        for (int g = 0; g < NG; ++g) sum.add(x[g].x), sum.add(x[g].y), sum.add(x[g].z), sum.add(x[g].w);
        S = sum.units();
    }
    int NF = 0;  // non-finite elements
    const bool finite = __all(squares < 0x7f800000u);
    if (!finite) {  // one by one, from memory again
        double part = 0.0;
#pragma unroll 1
        for (int c = threadIdx.x; 8 * c < K; c += NT)
#pragma unroll 1
            for (int k = 8 * c; k < 8 * c + 8 && k < K; ++k) {
                const uint16_t h = row[k];
                const bool fin = (h & 0x7c00) != 0x7c00;
                part += (double)(fin ? half_bits_to_float(h) : 0.0f);
                NF += fin ? 0 : 1;
            }
        S = double_units(part);
    }
    wave_sums<NT>(S, NF, s_mean);
    if constexpr (NT > 64) __syncthreads();
    row_sums<NT>(S, NF, s_mean);
    NF = K - NF;  // finite elements of the row
    // ceil(S / K): the quotient in double is off by less than one, its remainder says which way
    long long q = (long long)floor((double)S / (double)K);
    long long r = S - q * K;
    if (r < 0) --q, r += K;
    if (r >= K) ++q, r -= K;
    const float bound = half_grid_ceil(q + (r > 0 ? 1 : 0));
    const _Float16 bound16 = (_Float16)bound;  // exact
    uint16_t bbits;
    __builtin_memcpy(&bbits, &bound16, 2);
    const uint32_t bound2 = bbits * 0x10001u, one2 = 0x00010001u;
    // The second pass works on the registers again: kept opaque here, or the compiler carries what the
    // first one derived from them across the reduction.
#pragma unroll
    for (int g = 0; g < NG; ++g) asm volatile("" : "+v"(x[g].x), "+v"(x[g].y), "+v"(x[g].z), "+v"(x[g].w));

    int NN = 0;
    long long SN;
    uint32_t *dst = wsign + n * rw;
    auto finish = [&](int c, uint32_t bits) {
        const int left = K - 8 * c;  // elements from here to the row's end
        if (8 * NT * NG > K) bits &= (1u << (left >= 8 ? 8 : (left > 0 ? left : 0))) - 1u;  // +0 was loaded beyond it
        NN += __popc(bits);
        const uint32_t word = quad_word(bits, lane);  // whole quads stay together: rw is a multiple of 4
        if (c < 4 * rw && (lane & 3) == 0) dst[c >> 2] = word;
    };
    // the signs of the registers' groups; low(w) gets each group's elements below the bound, the others zero
    auto signs = [&](auto low) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            uint32_t w[4] = {x[g].x, x[g].y, x[g].z, x[g].w};
            uint32_t V = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t d, flag, keep;
                asm("v_pk_add_f16 %0, %1, %2 neg_lo:[0,1] neg_hi:[0,1] clamp" : "=v"(d) : "v"(bound2), "v"(w[i]));
                asm("v_pk_min_u16 %0, %1, %2" : "=v"(flag) : "v"(d), "v"(one2));  // 1 where x < bound
                asm("v_pk_sub_i16 %0, 0, %1" : "=v"(keep) : "v"(flag));           // 0xffff there
                V = flag << (2 * i) | V;
                w[i] &= keep;
            }
            low(w);
            int c = (int)threadIdx.x + NT * g;
            asm volatile("" : "+v"(c));  // its conditions are evaluated here, not carried through the kernel
            finish(c, (V & 0x55u) | (V >> 15 & 0xaau));
        }
    };
    if (small) {
        SmallSum low;
        signs([&](const uint32_t (&w)[4]) { low.add(w); });
        SN = low.units;
    } else if (finite) {
        SignedSum low;
        signs([&](const uint32_t (&w)[4]) { low.add(w[0]), low.add(w[1]), low.add(w[2]), low.add(w[3]); });
        SN = low.units();
    } else {
        double low = 0.0;
#pragma unroll 1
        for (int c = threadIdx.x; c < NT * NG; c += NT) {
            uint32_t bits = 0;
#pragma unroll 1
            for (int i = 0; i < 8 && 8 * c + i < K; ++i) {
                const uint16_t h = row[8 * c + i];
                const float f = half_bits_to_float(h);
                const bool neg = !(f >= bound);  // NaN and -Inf -> -1, +Inf -> +1
                const bool fin_neg = neg && (h & 0x7c00) != 0x7c00;
                bits |= (uint32_t)neg << i;
                low += (double)(fin_neg ? f : 0.0f);
                NN -= neg && !fin_neg ? 1 : 0;  // counted with the others
            }
            finish(c, bits);
        }
        SN = double_units(low);
    }
    wave_sums<NT>(SN, NN, s_below);
    if constexpr (NT > 64) __syncthreads();
    if (threadIdx.x == 0) {
        row_sums<NT>(SN, NN, s_below);
        const double T = (double)K * (double)(S - 2 * SN) - (double)S * (double)(NF - 2 * NN);
        s_w[n] = double_to_half_bits(T / ((double)K * (double)K * 16777216.0));
    }
}

// The same with RB rows to a workgroup of NW wavefronts: 64 / RB lanes of a wavefront hold that many groups of 8 consecutive
// elements of a row.  What a row costs whatever its length (two 64-bit reductions, two divisions in double, a search on
// the binary16 grid: some 200 instructions) is then spent on RB rows at a time and its divisions by one lane per row, where
// before every wavefront of every row went through all of it.  us replayed, before / after: 4096 x 768 5.1 / 4.4, 11008 x
// 1000 9.5 / 8.0, 11008 x 3000 18.8 / 15.3, 64 x 3000 4.3 / 3.8, 4096 x 5000 15.3 / 12.7, 5504 x 6000 19.2 / 15.5 (4.8 TB/s).  Four
// wavefronts: with eight 3 to 15 % slower, with one row per workgroup 20 % and more.
template <int RB, int NW, int NG>
__global__ __launch_bounds__(64 * NW) void k_prepare_weights_rows(const uint16_t *__restrict__ W, int64_t ldw, int N, int K, int rw,
                                                                 uint32_t *__restrict__ wsign, uint16_t *__restrict__ s_w)
{
    constexpr int LPR = 64 / RB;
    __shared__ long long s_sum[NW][RB], s_low[NW][RB], s_row[RB];
    __shared__ int s_bad[NW][RB], s_below[NW][RB], s_finite[RB];
    __shared__ uint32_t s_bound[RB];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane / LPR, cl = lane % LPR;
    const int64_t n = (int64_t)RB * blockIdx.x + r;
    const uint16_t *row = W + (n < N ? n : N - 1) * ldw;  // rows past the last: that one again, not stored
    const int first = LPR * wave + cl;
    constexpr int STEP = LPR * NW;
    uint4 x[NG];
    load_row<NG>(row, first, STEP, K, x);

    uint32_t squares = 0;  // the largest sum of a group's squares, as its bits
    SmallSum small_sum;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const uint32_t w[4] = {x[g].x, x[g].y, x[g].z, x[g].w};
        small_sum.add(w);
        float sq = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) sq = add_squares(w[i], sq);
        squares = max(squares, __float_as_uint(sq));
    }
    const bool small = __all(SmallSum::exact_below(squares));
    const bool finite = __all(squares < 0x7f800000u);
    long long S = small_sum.units;
    int bad = 0;  // non-finite elements
    if (!small) {
        if (finite) {
            SignedSum sum;
#pragma unroll
            for (int g = 0; g < NG; ++g) sum.add(x[g].x), sum.add(x[g].y), sum.add(x[g].z), sum.add(x[g].w);
            S = sum.units();
        } else {  // one by one, from memory again
            double part = 0.0;
#pragma unroll 1
            for (int c = first; 8 * c < K; c += STEP)
#pragma unroll 1
                for (int k = 8 * c; k < 8 * c + 8 && k < K; ++k) {
                    const uint16_t h = row[k];
                    const bool fin = (h & 0x7c00) != 0x7c00;
                    part += (double)(fin ? half_bits_to_float(h) : 0.0f);
                    bad += fin ? 0 : 1;
                }
            S = double_units(part);
            bad = lane_group_sum<LPR>(bad);
        }
    }
    S = lane_group_sum<LPR>(S);
    if (cl == 0) s_sum[wave][r] = S, s_bad[wave][r] = bad;
    __syncthreads();
    if (threadIdx.x < RB) {  // one lane per row
        long long T = 0;
        int b = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) T += s_sum[i][threadIdx.x], b += s_bad[i][threadIdx.x];
        // ceil(T / K): the quotient in double is off by less than one, its remainder says which way
        long long q = (long long)floor((double)T / (double)K);
        long long rem = T - q * K;
        if (rem < 0) --q, rem += K;
        if (rem >= K) ++q, rem -= K;
        const _Float16 bound16 = (_Float16)half_grid_ceil(q + (rem > 0 ? 1 : 0));  // exact
        uint16_t bbits;
        __builtin_memcpy(&bbits, &bound16, 2);
        s_bound[threadIdx.x] = bbits * 0x10001u, s_row[threadIdx.x] = T, s_finite[threadIdx.x] = K - b;
    }
    __syncthreads();
    const uint32_t bound2 = s_bound[r], one2 = 0x00010001u;
    // The second pass works on the registers again: kept opaque here, or the compiler carries what the
    // first one derived from them across the reduction.
#pragma unroll
    for (int g = 0; g < NG; ++g) asm volatile("" : "+v"(x[g].x), "+v"(x[g].y), "+v"(x[g].z), "+v"(x[g].w));

    int NN = 0;
    long long SN;
    uint32_t *dst = wsign + (n < N ? n : 0) * rw;
    const int words = n < N ? rw : 0;
    auto finish = [&](int c, uint32_t bits) {
        const int left = K - 8 * c;  // elements from here to the row's end
        if (8 * STEP * NG > K) bits &= (1u << (left >= 8 ? 8 : (left > 0 ? left : 0))) - 1u;  // +0 was loaded beyond it
        NN += __popc(bits);
        const uint32_t word = quad_word(bits, lane);  // whole quads stay together: rw is a multiple of 4
        if ((lane & 3) == 0 && (c >> 2) < words) dst[c >> 2] = word;
    };
    // the signs of the registers' groups; low(w) gets each group's elements below the bound, the others zero
    auto signs = [&](auto low) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            uint32_t w[4] = {x[g].x, x[g].y, x[g].z, x[g].w};
            uint32_t V = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t d, flag, keep;
                asm("v_pk_add_f16 %0, %1, %2 neg_lo:[0,1] neg_hi:[0,1] clamp" : "=v"(d) : "v"(bound2), "v"(w[i]));
                asm("v_pk_min_u16 %0, %1, %2" : "=v"(flag) : "v"(d), "v"(one2));  // 1 where x < bound
                asm("v_pk_sub_i16 %0, 0, %1" : "=v"(keep) : "v"(flag));           // 0xffff there
                V = flag << (2 * i) | V;
                w[i] &= keep;
            }
            low(w);
            int c = first + STEP * g;
            asm volatile("" : "+v"(c));  // its conditions are evaluated here, not carried through the kernel
            finish(c, (V & 0x55u) | (V >> 15 & 0xaau));
        }
    };
    if (small) {
        SmallSum low;
        signs([&](const uint32_t (&w)[4]) { low.add(w); });
        SN = low.units;
    } else if (finite) {
        SignedSum low;
        signs([&](const uint32_t (&w)[4]) { low.add(w[0]), low.add(w[1]), low.add(w[2]), low.add(w[3]); });
        SN = low.units();
    } else {
        const float bound = half_bits_to_float((uint16_t)bound2);
        double low = 0.0;
#pragma unroll 1
        for (int c = first; c < STEP * NG; c += STEP) {
            uint32_t bits = 0;
#pragma unroll 1
            for (int i = 0; i < 8 && 8 * c + i < K; ++i) {
                const uint16_t h = row[8 * c + i];
                const float f = half_bits_to_float(h);
                const bool neg = !(f >= bound);  // NaN and -Inf -> -1, +Inf -> +1
                const bool fin_neg = neg && (h & 0x7c00) != 0x7c00;
                bits |= (uint32_t)neg << i;
                low += (double)(fin_neg ? f : 0.0f);
                NN -= neg && !fin_neg ? 1 : 0;  // counted with the others
            }
            finish(c, bits);
        }
        SN = double_units(low);
    }
    SN = lane_group_sum<LPR>(SN);
    NN = lane_group_sum<LPR>(NN);
    if (cl == 0) s_low[wave][r] = SN, s_below[wave][r] = NN;
    __syncthreads();
    if (threadIdx.x < RB && (int64_t)RB * blockIdx.x + threadIdx.x < N) {
        SN = 0, NN = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) SN += s_low[i][threadIdx.x], NN += s_below[i][threadIdx.x];
        const long long T = s_row[threadIdx.x];
        const double sum = (double)K * (double)(T - 2 * SN) - (double)T * (double)(s_finite[threadIdx.x] - 2 * NN);
        s_w[(int64_t)RB * blockIdx.x + threadIdx.x] = double_to_half_bits(sum / ((double)K * (double)K * 16777216.0));
    }
}

// The same scale and, from the same registers, the ternarised row: one pass over A where
// bwta_act_scale followed by bwta_prepare_act makes two.  One workgroup of NT threads per row, for
// the two bit planes and for fragments of rows that k_act_scale_fragments cannot hold.  FRAG: E2M1
// fragments for the tiled matrix-core kernel (the grid also covers the padding rows of the last row
// blocks, and the threads the padding k steps: they write the zeros the product relies on).
// Thread t's group g is elements 8 (t + NT g) ..: the four lanes of a hardware quad hold one
// 32-element plane word, which both output forms assemble inside the quad.
template <int NG, int NT, bool FRAG>
__global__ __launch_bounds__(NT) void k_act_scale_quantize(const uint16_t *__restrict__ A, int64_t lda, int M, int K,
                                                           int rw, uint16_t *__restrict__ s_out,
                                                           uint32_t *__restrict__ frag, int s_pad,
                                                           uint32_t *__restrict__ mask, uint32_t *__restrict__ sign)
{
    __shared__ long long s_ll[NT / 64];
    const int m = blockIdx.x;
    const uint16_t *row = A + (int64_t)(m < M ? m : M - 1) * lda;
    uint4 x[NG];
    load_row<NG>(row, threadIdx.x, NT, K, x);
    const long long part = lane_group_sum<64>(magnitude_units(x));
    if ((threadIdx.x & 63) == 0) s_ll[threadIdx.x >> 6] = part;
    __syncthreads();
    long long S = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) S += s_ll[i];
    const uint16_t s_bits = m < M ? scale_bits(S, K) : (uint16_t)0;  // 0: an invalid scale, the row ternarises to zero
    if (threadIdx.x == 0 && m < M) s_out[m] = s_bits;
    // an all-zero (or all non-finite) row has s = 0, an invalid scale: the row ternarises to zero
    const TernaryThr thr = ternary_thresholds(s_bits, true);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int c = (int)threadIdx.x + NT * g, q = c >> 2, j = c & 3;
        if (FRAG) {
            const uint32_t D = fragment_dword(x[g], thr, j);
            int step, half;
            word_slot(q, step, half);
            if (step < s_pad)
                frag[(((int64_t)(m >> 5) * s_pad + step) * 64 + half * 32 + (m & 31)) * 4 + j] = D;
        } else {
            uint32_t nz, neg;
            ternary_flags<false>(x[g], thr, nz, neg);
            const uint32_t mw = quad_word(nz, lane), sw = quad_word(neg, lane);
            if (q < rw && j == 0) {
                mask[(int64_t)m * rw + q] = mw;
                sign[(int64_t)m * rw + q] = sw;
            }
        }
    }
}

// Scale and fragments in one pass (K <= 16384).  Bound: HBM (2 bytes in, half a byte out per element), with the
// vector ALU close behind (8.5 instructions per element).  A workgroup of NW wavefronts takes RB rows: a
// fragment holds 16 bytes per row with consecutive rows side by side, so a workgroup per row writes 16-byte
// pieces of lines that eight workgroups on eight XCDs share.  64 / RB lanes of a wavefront hold that many
// groups of 8 consecutive elements of a row, all NG loads of a thread are in flight before the first sum, and the
// row sums meet in LDS once.  Four rows (8 are within 10 %) where they still make 192 workgroups or more, as rows come
// in padded to 256: up to 512 rows two, up to 256 one, unless K is so short that launches are all there is.
// Two as well between K = 11265 and 12288, where four would run with a quarter of their lanes idle.
// us, a workgroup of 256 or 1024 threads per row with conversions to double before / four / two / one rows:
//    256 x  4096   3.8 / 4.0 / 3.6 / 3.4      512 x  4096   4.4 / 4.0 / 3.7 / 4.2
//    256 x 12288   5.9 / 8.0 / 4.8 / 4.7      512 x 12288   8.5 / 8.3 / 5.5 / 6.7
//   1024 x  4096   6.0 / 4.2 / 4.6 / 5.8     2048 x 11008  18.3 / 13.6 / 13.5 / 17.0 (4.1 TB/s)
template <int RB, int NW, int NG>
__global__ __launch_bounds__(64 * NW) void k_act_scale_fragments(const uint16_t *__restrict__ A, int64_t lda, int M,
                                                                int K, uint16_t *__restrict__ s_out,
                                                                uint32_t *__restrict__ frag, int s_pad)
{
    constexpr int LPR = 64 / RB;  // lanes, and groups of 8 elements, per row in one pass of a wavefront
    __shared__ long long s_part[NW][RB];
    __shared__ uint16_t s_bits[RB];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane / LPR, cl = lane % LPR, j = lane & 3;
    const int m = RB * blockIdx.x + r;
    uint4 x[NG];
    load_row<NG>(A + (int64_t)(m < M ? m : M - 1) * lda, LPR * wave + cl, LPR * NW, K, x);
    const long long part = lane_group_sum<LPR>(magnitude_units(x));
    if (cl == 0) s_part[wave][r] = part;
    __syncthreads();
    if (threadIdx.x < RB) {  // one division per row
        long long S = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) S += s_part[i][threadIdx.x];
        const int mt = RB * blockIdx.x + (int)threadIdx.x;
        const uint16_t b = mt < M ? scale_bits(S, K) : (uint16_t)0;  // 0: padding rows ternarise to zero
        s_bits[threadIdx.x] = b;
        if (mt < M) s_out[mt] = b;
    }
    __syncthreads();
    const TernaryThr thr = ternary_thresholds(s_bits[r], true);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        int step, half;
        word_slot((LPR * (NW * g + wave) + cl) >> 2, step, half);
        const uint32_t D = fragment_dword(x[g], thr, j);
        if (step < s_pad) frag[(((int64_t)(m >> 5) * s_pad + step) * 64 + half * 32 + (m & 31)) * 4 + j] = D;
    }
}

// mask plane of a binary (+-1) activation matrix: every element is non-zero; pad bits stay zero
__global__ __launch_bounds__(kThreads) void k_full_mask(uint32_t *__restrict__ mask, int64_t words, int rw, int K)
{
    const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (gid >= words) return;
    const int q = (int)(gid % rw), left = K - 32 * q;
    mask[gid] = left >= 32 ? 0xffffffffu : (left > 0 ? (1u << left) - 1u : 0u);
}

}  // namespace

hipError_t launch_full_mask(uint32_t *mask, int M, int K, hipStream_t st)
{
    const int rw = 4 * ((K + 127) / 128);
    const int64_t words = (int64_t)M * rw;
    if (words == 0) return hipSuccess;
    hipLaunchKernelGGL(k_full_mask, dim3((unsigned)((words + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, mask,
                       words, rw, K);
    return hipGetLastError();
}

hipError_t launch_prepare_weights(const void *W, int64_t ldw, int N, int K, uint32_t *wsign, uint16_t *s_w,
                                  hipStream_t st)
{
    if (N == 0) return hipSuccess;
    const int rw = 4 * ((K + 127) / 128);
    const int c8 = rw * 4;  // 128-bit groups per row; K <= 32768 -> at most 4096
#define BWTA_PREP(NG_, NT_)                                                                                   \
    if (c8 <= NG_ * NT_) {                                                                                    \
        hipLaunchKernelGGL((k_prepare_weights<NG_, NT_>), dim3(N), dim3(NT_), 0, st, (const uint16_t *)W, ldw, K, rw, \
                           wsign, s_w);                                                                       \
        return hipGetLastError();                                                                             \
    }
    // Rows side by side in a workgroup where the fixed part of a row counts (k_prepare_weights_rows): up to K = 2048 where
    // they are many, to 3072, and from 4097 to 6144; in between and beyond the registers of long rows decide, and the two
    // are level (4096 x 11008 20.8 / 20.7).
#define BWTA_PREPR(RB_, NG_)                                                                                             \
    if (c8 <= 64 / RB_ * 4 * NG_) {                                                                                      \
        hipLaunchKernelGGL((k_prepare_weights_rows<RB_, 4, NG_>), dim3((N + RB_ - 1) / RB_), dim3(256), 0, st,           \
                           (const uint16_t *)W, ldw, N, K, rw, wsign, s_w);                                              \
        return hipGetLastError();                                                                                        \
    }
    if (c8 <= 256 && N >= 2560) {
        BWTA_PREPR(4, 1) BWTA_PREPR(4, 2) BWTA_PREPR(4, 3) BWTA_PREPR(4, 4)
    }
    if (c8 > 256 && c8 <= 384) {
        if (N < 2048) {
            BWTA_PREPR(2, 3)
        }
        BWTA_PREPR(4, 6)
    }
    if (c8 > 512 && c8 <= 768 && N >= 896) {
        BWTA_PREPR(2, 6)
    }
#undef BWTA_PREPR
    BWTA_PREP(1, 64) BWTA_PREP(2, 64) BWTA_PREP(4, 64) BWTA_PREP(8, 64)
    BWTA_PREP(4, 256) BWTA_PREP(6, 256) BWTA_PREP(8, 256) BWTA_PREP(16, 256)
#undef BWTA_PREP
    return hipErrorInvalidValue;
}

hipError_t launch_act_scale(const void *A, int64_t lda, int M, int K, uint16_t *s, hipStream_t st)
{
    if (M == 0) return hipSuccess;
    const int c8 = (K + 7) / 8;  // K <= 32768 -> at most 4096
    // A wavefront per 64 / L rows up to 64 x 8 groups: beyond that the row would need more than 8 loads per
    // lane and too few wavefronts would share a row's latency.  Rows shorter than a load are read element by
    // element, one set of rows per wavefront (16 rows of 5: four sets 3.4 us, one 2.3).
#define BWTA_SCALE_W(L_, NG_, R_)                                                                              \
    if (c8 <= L_ * NG_) {                                                                                      \
        const int64_t rows_per_wg = (kThreads / 64) * (64 / L_) * R_;                                          \
        hipLaunchKernelGGL((k_act_scale_wave<L_, NG_, R_>), dim3((unsigned)((M + rows_per_wg - 1) / rows_per_wg)), \
                           dim3(kThreads), 0, st, (const uint16_t *)A, lda, M, K, s);                          \
        return hipGetLastError();                                                                              \
    }
    if (K < 8) {
        BWTA_SCALE_W(8, 1, 1)
    }
    BWTA_SCALE_W(8, 1, 4) BWTA_SCALE_W(16, 1, 4) BWTA_SCALE_W(32, 1, 4) BWTA_SCALE_W(64, 1, 4)
    if (M > 512) {
        BWTA_SCALE_W(64, 2, 2) BWTA_SCALE_W(64, 4, 1) BWTA_SCALE_W(64, 8, 1)
    }
#undef BWTA_SCALE_W
#define BWTA_SCALE(NG_, NT_)                                                                                       \
    if (c8 <= NG_ * NT_) {                                                                                         \
        hipLaunchKernelGGL((k_act_scale<NG_, NT_>), dim3(M), dim3(NT_), 0, st, (const uint16_t *)A, lda, K, s);    \
        return hipGetLastError();                                                                                  \
    }
    BWTA_SCALE(1, 256) BWTA_SCALE(2, 256) BWTA_SCALE(4, 256) BWTA_SCALE(6, 256) BWTA_SCALE(8, 256) BWTA_SCALE(16, 256)
#undef BWTA_SCALE
    return hipErrorInvalidValue;
}

// scale + ternarised operand in one pass; frag != nullptr selects fragments, else planes
hipError_t launch_act_scale_quantize(const void *A, int64_t lda, int M, int K, uint16_t *s_out, uint32_t *frag,
                                     uint32_t *mask, uint32_t *sign, hipStream_t st)
{
    if (M == 0) return hipSuccess;
    const int rw = 4 * ((K + 127) / 128);
    const int s_pad = fp4_s_pad(rw);
    const int rows = frag ? 32 * fp4_rb_pad(M) : M;
    const int c8 = frag ? 8 * s_pad : 4 * rw;  // 128-bit groups a row's threads must cover (padding included)
#define BWTA_SF(RB_, NW_, NG_)                                                                                     \
    if (c8 <= 64 / RB_ * NW_ * NG_) {                                                                              \
        hipLaunchKernelGGL((k_act_scale_fragments<RB_, NW_, NG_>), dim3(rows / RB_), dim3(64 * NW_), 0, st,         \
                           (const uint16_t *)A, lda, M, K, s_out, frag, s_pad);                                    \
        return hipGetLastError();                                                                                  \
    }
    // Rows per workgroup: see k_act_scale_fragments.  rows is a multiple of 256, c8 of 64.
    if (frag) {
        if (rows <= 256 && c8 > 128) {
            BWTA_SF(1, 4, 1) BWTA_SF(1, 8, 1) BWTA_SF(1, 8, 2) BWTA_SF(1, 8, 3) BWTA_SF(1, 8, 4)
        }
        if ((rows <= 512 && c8 > 64) || (c8 > 1408 && c8 <= 1536)) {
            BWTA_SF(2, 4, 1) BWTA_SF(2, 4, 2) BWTA_SF(2, 4, 4) BWTA_SF(2, 8, 4) BWTA_SF(2, 8, 6) BWTA_SF(2, 8, 8)
        }
        BWTA_SF(4, 4, 1) BWTA_SF(4, 4, 2) BWTA_SF(4, 4, 4) BWTA_SF(4, 8, 4) BWTA_SF(4, 8, 6) BWTA_SF(4, 8, 8)
        BWTA_SF(4, 8, 11) BWTA_SF(4, 8, 16)
    }
#undef BWTA_SF
    if (frag) {
        if (c8 > 4096) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_act_scale_quantize<4, 1024, true>), dim3(rows), dim3(1024), 0, st, (const uint16_t *)A, lda,
                           M, K, rw, s_out, frag, s_pad, mask, sign);
        return hipGetLastError();
    }
#define BWTA_SQ(NG_, NT_)                                                                                          \
    if (c8 <= NG_ * NT_) {                                                                                         \
        hipLaunchKernelGGL((k_act_scale_quantize<NG_, NT_, false>), dim3(rows), dim3(NT_), 0, st,                   \
                           (const uint16_t *)A, lda, M, K, rw, s_out, frag, s_pad, mask, sign);                    \
        return hipGetLastError();                                                                                  \
    }
    BWTA_SQ(1, 256) BWTA_SQ(2, 256) BWTA_SQ(4, 256) BWTA_SQ(8, 256) BWTA_SQ(4, 1024)
#undef BWTA_SQ
    return hipErrorInvalidValue;
}

hipError_t launch_quantize_pack(const void *A, int dtype, int64_t lda, ScaleArg s_a, int M, int K,
                                uint32_t *mask, uint32_t *sign, int32_t *nnz, hipStream_t st)
{
    const int rw = 4 * ((K + 127) / 128);
    const int64_t total = (int64_t)M * rw * 4;
    if (total == 0) return hipSuccess;
    const unsigned grid = (unsigned)((total + kThreads - 1) / kThreads);
    if (dtype == 0 && K >= 8 && (int64_t)M * rw >= kQuadGroupMinThreads)
        hipLaunchKernelGGL(k_quantize_pack_vec<0>, dim3((unsigned)(((int64_t)M * rw + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, st, (const uint16_t *)A, lda, s_a, M, K, rw, mask, sign);
    else if (dtype == 0)
        hipLaunchKernelGGL(k_quantize_pack<0>, dim3(grid), dim3(kThreads), 0, st, A, lda, s_a, M, K, rw,
                           mask, sign);
    else
        hipLaunchKernelGGL(k_quantize_pack<1>, dim3(grid), dim3(kThreads), 0, st, A, lda, s_a, M, K, rw,
                           mask, sign);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nnz == nullptr) return e;
    hipLaunchKernelGGL(k_row_popcount, dim3((M + 3) / 4), dim3(kThreads), 0, st, mask, M, rw, nnz);
    return hipGetLastError();
}

hipError_t launch_quantize_pack_bool(const void *A, int64_t lda, ScaleArg s_a, int M, int K, uint32_t *mask,
                                     hipStream_t st)
{
    const int rw = 4 * ((K + 127) / 128);
    const int64_t total = (int64_t)M * rw * 4;
    if (total == 0) return hipSuccess;
    const unsigned grid = (unsigned)((total + kThreads - 1) / kThreads);
    if (K >= 8 && (int64_t)M * rw >= kQuadGroupMinThreads)
        hipLaunchKernelGGL(k_quantize_pack_vec<2>, dim3((unsigned)(((int64_t)M * rw + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, st, (const uint16_t *)A, lda, s_a, M, K, rw, mask, (uint32_t *)nullptr);
    else
        hipLaunchKernelGGL(k_quantize_pack<2>, dim3(grid), dim3(kThreads), 0, st, A, lda, s_a, M, K, rw, mask,
                           (uint32_t *)nullptr);
    return hipGetLastError();
}

hipError_t launch_pack_weights(const void *W, int dtype, int64_t ldw, int N, int K, uint32_t *wsign,
                               hipStream_t st)
{
    const int rw = 4 * ((K + 127) / 128);
    const int64_t total = (int64_t)N * rw * 4;
    if (total == 0) return hipSuccess;
    const unsigned grid = (unsigned)((total + kThreads - 1) / kThreads);
    const int elt = dtype == 0 ? 2 : 1;
    const int vec_ok = (((uintptr_t)W % (8 * elt)) == 0 && (ldw % 8) == 0) ? 1 : 0;
    if (dtype == 0)
        hipLaunchKernelGGL(k_pack_weights<0>, dim3(grid), dim3(kThreads), 0, st, W, ldw, N, K, rw, wsign,
                           vec_ok);
    else
        hipLaunchKernelGGL(k_pack_weights<1>, dim3(grid), dim3(kThreads), 0, st, W, ldw, N, K, rw, wsign,
                           vec_ok);
    return hipGetLastError();
}

}  // namespace bwta
