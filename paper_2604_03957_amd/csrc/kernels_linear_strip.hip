// bwta_linear in one launch for K beyond what k_linear_fused holds at once: a workgroup owns 32 tokens x
// 128 NB channels and walks all of K in slabs of 512, ternarising the tokens' fp16 values on the way.
//
// Against ternarise + product the fragments are neither written nor read back and a launch with its ramp,
// first memory round trip and drain goes away; the price is that every workgroup of a token strip
// ternarises the strip again.  So it pays while the launch is one round of workgroups (see
// linear_strip_supported), where the two kernels are bound by latency and not by any unit.
//
//   * Eight wavefronts: four groups of channels x two halves of a slab (256 k each, summed through LDS at
//     the end; the sums are whole numbers, exact in fp32 in any order).
//   * A slab: every thread loads 4 groups of 8 activations (128-byte runs of a row) and NB 16-byte
//     pieces of weight rows (64-byte runs) two slabs ahead into registers, turns the activations into
//     matrix-core fragments and parks both in LDS for the next slab while the current one is multiplied
//     out of the other LDS stage: one barrier per slab.
//   * LDS: activation fragments in operand order, a step's kilobyte followed by 128 spare bytes (the two
//     words of a thread pair then lie in different banks); weight row r is its 64 bytes with piece c at
//     slot c ^ (r / 4 % 4), so that 16 neighbouring rows' 16-byte reads meet no bank twice.
//   * What bounds it: the vector ALU and the matrix cores in turn (two wavefronts per SIMD do not overlap
//     them fully): per slab 0.55 us of ternarising (31 instructions per 8 elements) and 0.25 NB of widening
//     weight bits and products; 3.4 to 5.2 us stand outside the slabs.  bwta_linear replayed back to back,
//     two kernels -> this one: 4096 x 768 x 3072 15.7 -> 12.8 us, 2048 x 768 x 2048 10.0 -> 8.1,
//     256 x 4096 x 4096 11.5 -> 10.5.  The loop copies no registers on purpose: with an exit between its two
//     slabs the compiler moved a requested slab at the back edge, waiting for all loads (6 % there).
#include <atomic>
#include <type_traits>

#include "bwta_internal.h"
#include "bwta_fp4_tile.h"

namespace bwta {

namespace {

template <int NB>
struct SCfg {
    static constexpr int BN = 128 * NB, THREADS = 512;
    static constexpr int A_STEP = 256 + 32, A_DW = 8 * A_STEP;  // dwords per step of 64 k, per slab
    static constexpr int W_DW = BN * 16;
    static constexpr int RED_DW = 4 * NB * 16 * 64;  // the second half's sums
    static constexpr int LOOP_DW = 2 * (A_DW + W_DW);
    static constexpr int WORK_DW = LOOP_DW > RED_DW ? LOOP_DW : RED_DW;
    static constexpr int SMEM_BYTES = (WORK_DW + 32 + BN) * 4;  // then [32] token scales, [BN] channel scales
    static_assert(32 * (32 * NB + 8) * 2 <= NB * 4096, "a wavefront's output strip lies where its sums were");
    static_assert(SMEM_BYTES <= 160 * 1024, "LDS of one compute unit");
};

template <int NB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void k_linear_strip(const uint16_t *__restrict__ A, int64_t lda, GemmArgs g, int tiles_n, int tiles_total)
{
    using C = SCfg<NB>;
    extern __shared__ __attribute__((aligned(1024))) uint32_t smem[];
    // ids are dealt to the 8 XCDs in turn; an XCD gets neighbouring tiles, channels fastest, so the tiles of
    // a strip find its activations in one L2
    int id;
    {
        const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3, chunk = tiles_total >> 3, rem = tiles_total & 7;
        id = xcd * chunk + (xcd < rem ? xcd : rem) + k;
    }
    const int m0 = 32 * (id / tiles_n), n0 = C::BN * (id % tiles_n);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, wn = wave & 3;  // half of the slab, group of channels
    const int r32 = lane & 31, h = lane >> 5;
    const int rw = g.rw;
    float *s_sa = (float *)(smem + C::WORK_DW), *s_sw = s_sa + 32;

    // ---- scales: requested first, parked before the first barrier
    const int row = (tid >> 3) & 31, j = tid & 3, m = m0 + row;
    const int mc = m < g.M ? m : 0;
    const bool have_sa = g.s_a.mode != 0 && g.s_a.ptr != nullptr, have_sw = g.s_w.mode != 0 && g.s_w.ptr != nullptr;
    const uint16_t sa_bits = *(have_sa ? g.s_a.ptr + (g.s_a.mode == 1 ? 0 : mc) : A);
    const bool want_sw = tid < C::BN && n0 + tid < g.N;
    const uint16_t sw_bits = *(want_sw && have_sw ? g.s_w.ptr + (g.s_w.mode == 1 ? 0 : n0 + tid) : A);

    // ---- what this thread loads: of words 4 it + q0 of a slab its 8 activations of `row`; pieces tid & 3 of
    // weight rows tid / 4 + 128 i.  Loads beyond the rows' end re-read the end (their products meet zero
    // activations), rows beyond the matrix another row (ternarised to zero, or never stored).
    const uint16_t *a_row = A + (int64_t)mc * lda;
    const int q0 = 2 * (tid >> 8) + ((tid >> 2) & 1);
    const uint32_t *w_row[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int n = n0 + (tid >> 2) + 128 * i;
        w_row[i] = g.wsign + (int64_t)(n < g.N ? n : g.N - 1) * rw;
    }
    struct Slab {
        uint4 x[4], w[NB];
    };
    auto request = [&](Slab &s, int c) {
#pragma unroll
        for (int it = 0; it < 4; ++it) s.x[it] = request_group(a_row, 32 * (16 * c + 4 * it + q0) + 8 * j, g.K);
        int kw = 16 * c + 4 * (tid & 3);
        kw = kw < rw ? kw : rw - 4;
#pragma unroll
        for (int i = 0; i < NB; ++i) s.w[i] = *(const uint4 *)(w_row[i] + kw);
    };

    const int nslab = (rw + 15) >> 4;
    Slab s0, s1;
    request(s0, 0);
    request(s1, 1);
    __builtin_amdgcn_sched_barrier(0);

    const TernaryThr thr = ternary_thresholds(have_sa ? sa_bits : 0x3c00u, m < g.M);
    if ((tid & 263) == 0) s_sa[row] = m < g.M ? (have_sa ? half_bits_to_float(sa_bits) : 1.0f) : 0.0f;
    if (tid < C::BN) s_sw[tid] = want_sw ? (have_sw ? half_bits_to_float(sw_bits) : 1.0f) : 0.0f;

    auto park_a = [&](const Slab &s, int c, int stage, int it, auto end) {  // only the last slab reaches the rows' end
        const int q = 4 * it + q0, jw = q & 7;
        const uint4 x = decltype(end)::value ? finish_group(s.x[it], 32 * (16 * c + q) + 8 * j, g.K) : s.x[it];
        smem[stage * C::A_DW + (4 * (q >> 3) + (jw & 3)) * C::A_STEP + ((jw >> 2) * 32 + row) * 4 + j] = fragment_dword(x, thr, j);
    };
    auto park_w = [&](const Slab &s, int stage) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int r = (tid >> 2) + 128 * i;
            *(uint4 *)(smem + 2 * C::A_DW + stage * C::W_DW + 16 * r + 4 * ((tid & 3) ^ ((r >> 2) & 3))) = s.w[i];
        }
    };

    v16f acc[NB][1];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][0][v] = 0.0f;
    uint32_t m88 = 0x88888888u, c22 = 0x22222222u;
    asm volatile("" : "+s"(m88));
    asm volatile("" : "+v"(c22));

    const uint32_t *a_rd = smem + 4 * kg * C::A_STEP + 4 * lane;
    const uint32_t *w_rd = smem + 2 * C::A_DW + 16 * (32 * NB * wn + r32) + 4 * ((2 * kg + h) ^ ((r32 >> 2) & 3));
    // the four steps of a slab, whose LDS reads are all requested first; before(st) goes in front of step st
    auto multiply = [&](int stage, auto before) {
        uint4 wq[NB], av[4];
#pragma unroll
        for (int b = 0; b < NB; ++b) wq[b] = *(const uint4 *)(w_rd + stage * C::W_DW + 512 * b);
#pragma unroll
        for (int st = 0; st < 4; ++st) av[st] = *(const uint4 *)(a_rd + stage * C::A_DW + st * C::A_STEP);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            before(st);
            const v8i a = {(int)av[st].x, (int)av[st].y, (int)av[st].z, (int)av[st].w, 0, 0, 0, 0};
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const v8i w = widen_w(st == 0 ? wq[b].x : st == 1 ? wq[b].y : st == 2 ? wq[b].z : wq[b].w, m88, c22);
                acc[b][0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, a, acc[b][0], 4, 4, 0, 0, 0, 0);
            }
        }
    };

    park_w(s0, 0);
#pragma unroll
    for (int it = 0; it < 4; ++it) park_a(s0, 0, 0, it, std::false_type{});
    request(s0, 2);
    __syncthreads();
    // slab c is multiplied while slab c + 1 (in `next`, requested two slabs ago) is parked in the other stage,
    // which the barrier before this slab released
    auto slab = [&](int c, Slab &next, int stage, auto end) {
        multiply(stage, [&](int st) {
            if (st == 0) park_w(next, stage ^ 1);
            park_a(next, c + 1, stage ^ 1, st, end);
        });
        if (!decltype(end)::value) request(next, c + 3);
        __syncthreads();
    };
    constexpr std::false_type inner{};
    constexpr std::true_type last{};
    int c = 0;
    for (; c + 3 < nslab; c += 2) {
        slab(c, s1, 0, inner);
        slab(c + 1, s0, 1, inner);
    }
    if (c + 2 < nslab) {
        slab(c, s1, 0, inner);
        slab(c + 1, s0, 1, last);
    } else {
        slab(c, s1, 0, last);
    }
    multiply((nslab - 1) & 1, [](int) {});

    // ---- the second half's sums join the first's
    __syncthreads();
    float4 *red = (float4 *)smem + wn * (NB * 4 * 64) + lane;
    if (kg == 1) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                red[(4 * b + q) * 64] = make_float4(acc[b][0][4 * q], acc[b][0][4 * q + 1], acc[b][0][4 * q + 2], acc[b][0][4 * q + 3]);
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 o = red[(4 * b + q) * 64];
            acc[b][0][4 * q] += o.x, acc[b][0][4 * q + 1] += o.y, acc[b][0][4 * q + 2] += o.z, acc[b][0][4 * q + 3] += o.w;
        }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int n_wave = n0 + 32 * NB * wn;
    if (n_wave >= g.N) return;
    store_tile_fp16<1, NB>(acc, g, s_sa, s_sw + 32 * NB * wn, (uint16_t *)(smem + wn * (NB * 1024)), m0, n_wave, lane);
}

template <int NB>
hipError_t launch_t(const void *A, int64_t lda, const GemmArgs &g, hipStream_t st)
{
    using C = SCfg<NB>;
    if (C::SMEM_BYTES > 64 * 1024) {  // said once per device
        static std::atomic<uint64_t> configured{0};
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = 1ull << (dev & 63);
        if (!(configured.load(std::memory_order_relaxed) & bit)) {
            e = hipFuncSetAttribute((const void *)k_linear_strip<NB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    C::SMEM_BYTES);
            if (e != hipSuccess) return e;
            configured.fetch_or(bit, std::memory_order_relaxed);
        }
    }
    const int64_t tiles_n = ((int64_t)g.N + C::BN - 1) / C::BN, total = tiles_n * (((int64_t)g.M + 31) / 32);
    if (total > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_linear_strip<NB>, dim3((unsigned)total), dim3(C::THREADS), C::SMEM_BYTES, st, (const uint16_t *)A,
                       lda, g, (int)tiles_n, (int)total);
    return hipGetLastError();
}

}  // namespace

// Channel blocks of 32 per wavefront: the fewest that leave at most one workgroup per compute unit (a second
// round costs as much as the first), 0 where three do not.
static int strip_blocks(const GemmArgs &g)
{
    for (int nb = 1; nb <= 3; ++nb)
        if (((int64_t)g.M + 31) / 32 * (((int64_t)g.N + 128 * nb - 1) / (128 * nb)) <= 256) return nb;
    return 0;
}

// Where one launch is ahead.  Its time is about 3.4 / 4.0 / 5.2 us + 0.8 / 1.0 / 1.3 us per slab of 512 for NB = 1 / 2 /
// 3, whatever M and N; that of the two kernels grows with M K (ternarising, fragments out and in).  Measured on 900
// shapes, M 2 .. 8192, N 64 .. 28000, K 520 .. 30000, replayed from a graph, two kernels / one, us:
//   Up to 128 tokens (the decode kernel is the other side) level up to K = 1536 (64 x 768 5.8 / 5.6); at K = 2048
//   6 to 16 % behind with few outputs (64 x 768 5.9 / 6.5) but 10 to 20 % ahead where calls are made one by one (7.5 /
//   6.2), ahead with many (128 x 8192 8.3 / 7.1); beyond, up to 40 % behind and no faster call by call (64 x 768 x 3072
//   6.0 / 8.1, 7.9 / 7.8) except with many outputs: from a quarter of a million at K = 2560 (64 x 8192 x 2500 8.8 /
//   7.6), from half a million at K = 3072 (33 x 16384 9.3 / 8.5, 128 x 8192 9.5 / 8.3).
//   NB = 1 from 129 tokens ahead everywhere: 256 x 4096 x 2048 8.3 / 7.1, 256 x 4096 x 16384 31.8 / 30.0.
//   NB = 2 ahead from 513 tokens (513 x 3072 x 2048 9.1 / 8.2, 777 x 1536 x 4096 13.8 / 11.9), mixed below (512 x 4096 x
//   4096 12.3 / 11.9, 256 x 8192 x 4096 12.4 / 13.0); at K = 30000 only with narrow matrices (777 x 2500 63.9 / 71.6,
//   2048 x 768 78.6 / 68.5), whose tiles suit the other side less.
//   NB = 3 ahead from 2048 tokens (4096 x 768 x 3072 15.7 / 12.8, 2048 x 1536 x 2048 11.4 / 10.1), mixed below (777 x 3072 x
//   4096 15.3 / 14.2, 1024 x 3072 x 11008 28.3 / 32.0); beyond K = 8192 only with narrow matrices (2048 x 1536 x 11008 31.5 /
//   33.5, 4096 x 768 x 11008 39.1 / 33.2).
// From K = 3073 to 12288 the two kernels end in the product of 16 x 16 blocks with K split inside the workgroup, which
// leaves this kernel what is cheap to ternarise often or too narrow for it (strip_keeps_long_k; two kernels / one, us; up
// to K = 6144 shapes of at most 256 workgroups of 16 tokens x 128 channels are the strips of 16 tokens' and not meant):
//   NB = 1 up to K = 5120 (1024 x 1000 x 4096 12.1 / 10.3, 777 x 1152 x 4096 11.6 / 10.1, 512 x 2048 x 4096 10.6 / 10.0; few
//   tokens against wide matrices are behind, 256 x 4096 x 5000 11.8 / 13.1), to 7168 from 641 tokens (777 x 768 x 6500
//   16.1 / 14.4, 1500 x 600 x 6500 18.2 / 15.8; 512 x 2048 x 6000 12.0 / 14.2), beyond only tall and narrow
//   (2048 x 512 x 11008 23.6 / 22.7; 777 x 2048.. and wider behind, 256 x 4096 x 11008 16.4 / 21.9).  With an odd number of
//   pairs of slabs, 11 and 13 from 513 tokens (627 x 605 x 6576 15.1 / 13.9), 15 from 769 (1057 x 512 x 7236 17.1 / 15.9), 17
//   from 897 (1142 x 406 x 8478 19.1 / 18.1; 23 shapes in these windows 1.03 of its time).
//   NB = 2 up to K = 4608 for N <= 1536 (1300 x 1152 x 4096 14.4 / 13.9; 1024 x 2048 x 4096 13.2 / 14.3), to 7168 for N <= 768
//   (2048 x 768 x 5000 17.8 / 16.5; 777 x 1536 x 6000 14.2 / 16.3), beyond for N <= 512 (4096 x 512 x 11008 32.0 / 28.4; mixed at fewer tokens, 2221 x 407 x 9643 23.3 / 27.2).
//   NB = 3 beyond 8192 for N <= 768 (4096 x 768 x 11008 37.8 / 32.6; 2048 x 1152 x 11008 29.3 / 31.8).
// Longer K and N below 256 were not swept again.
static bool strip_keeps_long_k(const GemmArgs &g, int nb)
{
    if (g.K <= 3072 || g.K > 12288 || g.N < 256) return true;
    if (nb == 1) {
        const int pairs = (g.K + 511) / 512;  // odd: a group of wavefronts of the other kernel idles for one
        if (pairs % 2 == 1 && pairs <= 17 && g.M > (pairs <= 13 ? 512 : pairs == 15 ? 768 : 896)) return true;
        return g.K <= 5120 || (g.M > 640 && g.K <= 7168) || (g.M >= 1280 && g.N <= 512);
    }
    if (nb == 2) return g.N <= (g.K <= 4608 ? 1536 : g.K <= 7168 ? 768 : 512);
    return g.K <= 8192 || g.N <= 768;
}

bool linear_strip_supported(const GemmArgs &g)
{
    if (g.K <= 512 || g.out == nullptr || g.acc != nullptr || fp4_tuning_forced()) return false;
    const int nb = strip_blocks(g);
    const int64_t outputs = (int64_t)g.M * g.N;
    if (g.M <= 128)
        return (nb == 1 || nb == 2) &&
               (g.K <= 2048 || (g.K <= 2560 && outputs >= 256 * 1024) || (g.K <= 3072 && outputs > 512 * 1024));
    if (!strip_keeps_long_k(g, nb)) return false;
    const bool narrow = g.N <= 1152;
    return nb == 1 || (nb == 2 && g.M > 512 && (g.K <= 16384 || narrow)) || (nb == 3 && g.M >= 2048 && (g.K <= 8192 || narrow));
}

hipError_t launch_linear_strip(const void *A, int64_t lda, const GemmArgs &g, hipStream_t st)
{
    switch (strip_blocks(g)) {
    case 1: return launch_t<1>(A, lda, g, st);
    case 2: return launch_t<2>(A, lda, g, st);
    case 3: return launch_t<3>(A, lda, g, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace bwta
