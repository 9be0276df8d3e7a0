// BWTA product on the FP4 matrix cores in blocks of 16 x 16 (v_mfma_f32_16x16x128_f8f6f4, both operands
// E2M1): the kernel for long K.  Same operands, same exact sums as the kernels with blocks of 32 x 32
// (kernels_gemm_fp4.hip); other instruction, larger wavefront tiles, K split inside the workgroup.
//
//   * Why 16 x 16.  The clock of a large product drops under the power of toggling operands.  Per multiply-accumulate
//     this instruction updates its accumulators half as often as the 32 x 32 one: on random operands a loop of nothing
//     but MFMAs runs at 9.05 PFLOP/s and 2.26 GHz against 7.70 and 1.93 (on zeros both 9.84 at 2.4).  The weights are the
//     first operand (A first: 8.64), and the token blocks are walked there and back so that neighbouring instructions
//     share an operand (9.20).
//   * A wavefront owns 64 tokens x 128 channels: 32 blocks, 128 accumulators.  Its activation fragments come
//     straight from global memory (L2) into registers, four steps of 128 k ahead.  With one wavefront across the
//     channels (the tiles of 128) nobody else in the workgroup needs them; with two (128 x 256) both fetch them.
//     Lane (r16, q4) takes of a step the pieces (step q4 / 2, half q4 % 2) of its row in the fragment layout of the
//     32 x 32 kernels, four runs of 256 bytes per load.
//   * Weights, 1 bit each, go to LDS by direct loads for a pair of slabs (512 k, 64 bytes per channel) at a time,
//     one pair ahead, and from there to registers one step ahead of use.  A direct load lays lane l at 16 l, so the
//     four lanes of a row fetch its pieces in the order that leaves piece c of row r at slot c ^ (r / 4 % 4): the
//     4-byte reads of 16 neighbouring rows then meet no bank twice.  LDS reads are inline assembly with explicit
//     waits, through which the values pass: a read that the compiler sees makes it wait for every direct load.
//   * A block of 16 channels is widened (7 vector-ALU operations) between the four MFMAs on the block before it.
//     In one wavefront an MFMA and what follows it still take 23 clocks instead of 16; two wavefronts per SIMD fill
//     each other's gaps (0.95 of the matrix rate).  They fit by registers (236, KS = 2 246, of 256).
//   * KS groups of wavefronts in a workgroup take every KS-th pair of slabs, so that a compute unit has eight
//     wavefronts also where it gets one tile of 64 x KS.. outputs and not two; in the end every group keeps 64 / KS
//     tokens and hands the others' sums over through LDS, in fp32 (whole numbers, exact in any order).  Which
//     token blocks a group keeps is settled by the order in which it loads them, so the code is the same for all.
//   * Rows past the last arrive as zeros (buffer loads) and their results are not stored; words past a row's end are the
//     next row's and meet fragments of zeros.
//   * What bounds it now: waiting more than power.  Of the clocks that a compute unit is busy the matrix pipes are so for
//     67 % at 2048 x 4096 x 11008, 62 % at 2048 x 11008 x 4096, 51 % at 2048 x 4096 x 4096.  The first takes 33.9 us on
//     random operands at 1.9 GHz and 29.8 on zeros at 2.37, that is 4 us for the clock; its MFMAs are 19.0 us at 2.37
//     GHz, the time until the first one 1.5, the results 3.4 (5 TB/s): some 6 us are stalls of the loop.  With fragments
//     from one cache line instead of the L2 it takes 30.4, with weights that do not change 28.7.
//     us on ready fragments, random operands, the 32 x 32 kernels / this one: 2048 x 4096 x 4096 16.6 / 15.5 (KS = 2),
//     2048 x 4096 x 11008 38.4 / 34.3, 2048 x 11008 x 4096 40.9 / 38.2 (KS = 1), 512 x 4096 x 11008 15.6 / 13.7 (KS = 4).
//   * Tried: shifting the words of two channel blocks at once (v_lshlrev_b64: -1 % for KS = 2, +1 % for KS = 1); eight
//     wavefronts with KS = 2 on 256 x 128 (one workgroup per compute unit, no store under another's loop: 4 to 15 % slower
//     where tiles come to more than one round); the last partial round of tiles as K-split halves in the same launch
//     (level: what it saves in clocks the clock rate takes back).
#include <atomic>
#include <type_traits>

#include "bwta_internal.h"
#include "bwta_fp4_tile.h"

namespace bwta {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int RING = 4;          // k steps of 128 whose activation fragments are in flight or in use
constexpr int PITCH = 128 + 8;   // halfs per row of an output strip

template <int WAVES_M, int WAVES_N, int KS>
struct WCfg {
    static constexpr int BM = 64 * WAVES_M, BN = 128 * WAVES_N;
    static constexpr int NW = WAVES_M * WAVES_N, THREADS = 64 * NW * KS;
    static constexpr int W_ROUNDS = BN / 16 / NW;  // direct loads (16 channels, 1 KiB) per wavefront and pair of slabs
    static constexpr int W_BYTES = BN * 64;
    static constexpr int LOOP_BYTES = 2 * KS * W_BYTES;
    static constexpr int STRIP_BYTES = (KS == 4 ? 16 : 32) * PITCH * 2;
    static constexpr int RED_BYTES = 16 * 1024;  // what a wavefront hands to another: 64 accumulators
    // one group: the strips lie behind the stages; several: in what a wavefront has read of the others' sums
    static constexpr int STRIP_BASE = KS == 1 ? LOOP_BYTES : 0;
    static constexpr int STRIP_STEP = KS == 1 ? STRIP_BYTES : RED_BYTES;
    static constexpr int WORK_BYTES = KS == 1 ? LOOP_BYTES + NW * STRIP_BYTES
                                              : (LOOP_BYTES > NW * KS * RED_BYTES ? LOOP_BYTES : NW * KS * RED_BYTES);
    static constexpr int SMEM_BYTES = WORK_BYTES + (BN + BM) * 4;
    static_assert(BN / 16 % NW == 0, "every wavefront issues the same loads");
    static_assert(THREADS == 256 && SMEM_BYTES <= 80 * 1024, "two workgroups of four wavefronts per compute unit");
};

template <int WAVES_M, int WAVES_N, int KS>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * KS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_fp4_wide(GemmArgs g, const uint32_t *__restrict__ frag, int s_pad, int tiles_n, int tiles_total)
{
    using C = WCfg<WAVES_M, WAVES_N, KS>;
    extern __shared__ __attribute__((aligned(1024))) uint32_t smem[];
    int tm, tn;
    tile_of_workgroup(tiles_n, tiles_total, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KS == 1 ? 0 : wave / C::NW, wl = KS == 1 ? wave : wave % C::NW;
    const int wm = wl / WAVES_N, wn = wl % WAVES_N;
    const int r16 = lane & 15, q4 = lane >> 4;
    const int m0 = tm * C::BM, n0 = tn * C::BN;
    const int rw = g.rw;
    const int npair = s_pad >> 3, niter = (npair + KS - 1) / KS;

    // ---- weights of a pair of slabs (512 k), 64 bytes per channel, straight into LDS
    const auto w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)g.wsign, 0, (int)((uint32_t)g.N * (uint32_t)rw * 4u), 0x00020000);
    uint32_t w_off[C::W_ROUNDS];
#pragma unroll
    for (int q = 0; q < C::W_ROUNDS; ++q)
        w_off[q] = (uint32_t)(n0 + 16 * (q * C::NW + wl) + (lane >> 2)) * (uint32_t)rw * 4u + 16u * (uint32_t)((lane & 3) ^ (lane >> 4));
    // the pair a group takes in iteration it; past the end it asks for the last one again
    auto pair_of = [&](int it) { return it * KS + kg < npair ? it * KS + kg : npair - 1; };
    // the whole offset goes into the lane's address, which is what the range check looks at
    auto request_w = [&](int q, int it) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            w_rsrc, (void __attribute__((address_space(3))) *)(smem + ((2 * kg + (it & 1)) * C::W_BYTES) / 4 + (q * C::NW + wl) * 256), 16,
            (int)(w_off[q] + 64u * (uint32_t)pair_of(it)), 0, 0, 0);
    };
#pragma unroll
    for (int q = 0; q < C::W_ROUNDS; ++q) request_w(q, 0);

    constexpr int SW_PER = (C::BN + C::THREADS - 1) / C::THREADS, SA_PER = (C::BM + C::THREADS - 1) / C::THREADS;
    const uint16_t *scale_safe = (const uint16_t *)g.wsign;
    uint16_t sw_bits[SW_PER], sa_bits[SA_PER];
    const bool any_sw = g.s_w.mode != 0 && g.s_w.ptr != nullptr, any_sa = g.s_a.mode != 0 && g.s_a.ptr != nullptr;
#pragma unroll
    for (int i = 0; i < SW_PER; ++i) {
        const int e = tid + i * C::THREADS;
        sw_bits[i] = *(any_sw && e < C::BN && n0 + e < g.N ? g.s_w.ptr + (g.s_w.mode == 1 ? 0 : n0 + e) : scale_safe);
    }
#pragma unroll
    for (int i = 0; i < SA_PER; ++i) {
        const int e = tid + i * C::THREADS;
        sa_bits[i] = *(any_sa && e < C::BM && m0 + e < g.M ? g.s_a.ptr + (g.s_a.mode == 1 ? 0 : m0 + e) : scale_safe);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- activations, straight into registers.  Block i of 16 tokens is, of the wavefront's 64, the one whose bits are
    // i's xor the group's: every group keeps its first blocks in the end
    const auto a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)frag + (int64_t)(tm * (C::BM / 32) + wm * 2) * s_pad * 1024), 0,
                                                          2 * s_pad * 1024, 0x00020000);
    const int rb_flip = KS == 2 ? kg : KS == 4 ? kg >> 1 : 0, b_flip = KS == 4 ? kg & 1 : 0;
    const int a_lane = (q4 * 32 + r16) * 16 + 256 * b_flip, a_lane1 = a_lane ^ 256;
    const int a_blk0 = rb_flip * s_pad * 1024, a_blk1 = (rb_flip ^ 1) * s_pad * 1024;
    u32x4 ring[RING][4];
    auto load_a = [&](u32x4 &dst, int i, int it, int c) {
        dst = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (i & 1) ? a_lane1 : a_lane, (4 * pair_of(it) + c) * 2048 + ((i >> 1) ? a_blk1 : a_blk0), 0);
    };

    v4f acc[8][4];  // [block of 16 channels][block of 16 tokens]
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    uint32_t m88 = 0x88888888u, c22 = 0x22222222u;
    asm volatile("" : "+s"(m88));
    asm volatile("" : "+v"(c22));

#pragma unroll
    for (int s = 0; s < RING; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) load_a(ring[s][i], i, 0, s);
#pragma unroll
    for (int q = 0; q < C::W_ROUNDS; ++q) request_w(q, 1);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t *)smem;
    // lane (r16, q4) of a step takes word 0, 2, 1, 3 (q4 = 0 .. 3) of the row's four: the order the fragments have
    const uint32_t w_rd = lds0 + (uint32_t)(2 * kg * C::W_BYTES + (wn * 128 + r16) * 64 + ((r16 >> 2) & 3) * 16 + ((q4 & 1) * 2 + (q4 >> 1)) * 4);

    float *sc_lds = (float *)((char *)smem + C::WORK_BYTES);
#pragma unroll
    for (int i = 0; i < SW_PER; ++i) {
        const int e = tid + i * C::THREADS;
        if (e < C::BN) sc_lds[e] = n0 + e < g.N ? (any_sw ? half_bits_to_float(sw_bits[i]) : 1.0f) : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < SA_PER; ++i) {
        const int e = tid + i * C::THREADS;
        if (e < C::BM) sc_lds[C::BN + e] = m0 + e < g.M ? (any_sa ? half_bits_to_float(sa_bits[i]) : 1.0f) : 0.0f;
    }
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 * RING + C::W_ROUNDS) : "memory");
    __builtin_amdgcn_s_barrier();

    u32x2 wv[2][4];  // words of a step's 8 blocks of channels
    auto read_w = [&](u32x2 (&w)[4], int it, int c) {
        const uint32_t addr = (w_rd + (uint32_t)((it & 1) * C::W_BYTES)) ^ (uint32_t)(16 * c);
        asm volatile("ds_read2st64_b32 %0, %1 offset0:0 offset1:4" : "=v"(w[0]) : "v"(addr) : "memory");
        asm volatile("ds_read2st64_b32 %0, %1 offset0:8 offset1:12" : "=v"(w[1]) : "v"(addr) : "memory");
        asm volatile("ds_read2st64_b32 %0, %1 offset0:16 offset1:20" : "=v"(w[2]) : "v"(addr) : "memory");
        asm volatile("ds_read2st64_b32 %0, %1 offset0:24 offset1:28" : "=v"(w[3]) : "v"(addr) : "memory");
    };
    auto wait_w = [&](u32x2 (&w)[4]) {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3])::"memory");
    };
    v8i vb[2];
    auto widen_part = [&](v8i &v, uint32_t x, int d) { v[d] = (int)(((d < 3 ? x << (3 - d) : x) & m88) | c22); };
    // One step of 128 k.  Between the MFMAs on one block of channels the next block's operand is widened, behind the
    // last block's `after` asks for fragments.
    auto step = [&](const u32x4 (&a)[4], const u32x2 (&w)[4], u32x2 (&nw)[4], auto have_next, auto after) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j == 7 && decltype(have_next)::value) wait_w(nw);
            const v8i &cur = vb[j & 1];
            v8i &nxt = vb[(j + 1) & 1];
            const uint32_t x = j < 7 ? ((j + 1) & 1 ? w[(j + 1) >> 1].y : w[(j + 1) >> 1].x) : nw[0].x;
#pragma unroll
            for (int i0 = 0; i0 < 4; ++i0) {
                const int i = (j & 1) ? 3 - i0 : i0;  // there and back: neighbouring instructions share an operand
                const v8i va = {(int)a[i].x, (int)a[i].y, (int)a[i].z, (int)a[i].w, 0, 0, 0, 0};
                acc[j][i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(cur, va, acc[j][i], 4, 4, 0, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (j < 7 || decltype(have_next)::value) widen_part(nxt, x, i0);
                if (j == 7) after(i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    __builtin_amdgcn_s_setprio(3);
    read_w(wv[0], 0, 0);
    wait_w(wv[0]);
#pragma unroll
    for (int d = 0; d < 8; ++d) vb[0][d] = vb[1][d] = 0;
#pragma unroll
    for (int d = 0; d < 4; ++d) widen_part(vb[0], wv[0][0].x, d);
    auto pair_body = [&](int it, auto last) {
        constexpr bool LAST = decltype(last)::value;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c < 3) {
                read_w(wv[(c + 1) & 1], it, c + 1);
            } else if (!LAST) {
                // this pair's words have all been read (waited for in the step before); the next pair's own requests
                // are older than the 12 fragment loads of this pair's steps.  The count holds while nothing else of this
                // wavefront reaches memory here: a spilled register's store or reload would be counted too and the
                // words read too early, so the kernel must not use scratch (the tests look at the compiler's report)
                asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                read_w(wv[0], it + 1, 0);
#pragma unroll
                for (int q = 0; q < C::W_ROUNDS; ++q) request_w(q, it + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (c < 3 || !LAST)
                step(ring[c], wv[c & 1], wv[(c + 1) & 1], std::true_type{}, [&](int i) { if (!LAST) load_a(ring[c][i], i, it + 1, c); });
            else
                step(ring[c], wv[c & 1], wv[(c + 1) & 1], std::false_type{}, [](int) {});
        }
    };
    for (int it = 0; it + 1 < niter; ++it) pair_body(it, std::false_type{});
    if (KS == 1 || (niter - 1) * KS + kg < npair) pair_body(niter - 1, std::true_type{});
    __builtin_amdgcn_s_setprio(0);
    // pairs past the end are requested as well (never read): nothing may reach LDS behind this wavefront's back
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // ---- the groups' sums (whole numbers, exact in fp32 in any order)
    char *mine = (char *)smem + C::STRIP_BASE + wave * C::STRIP_STEP;
    if constexpr (KS > 1) {
        __builtin_amdgcn_s_barrier();
        auto exchange = [&](int partner, auto keep) {  // blocks keep .. 2 keep - 1 go to the partner
            constexpr int KEEP = decltype(keep)::value;
            v4f *dst = (v4f *)((char *)smem + partner * C::RED_BYTES) + lane, *src = (v4f *)mine + lane;
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int i = 0; i < KEEP; ++i) dst[(j * KEEP + i) * 64] = acc[j][KEEP + i];
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int i = 0; i < KEEP; ++i) acc[j][i] += src[(j * KEEP + i) * 64];
        };
        exchange(wave ^ (KS == 2 ? C::NW : 2 * C::NW), std::integral_constant<int, 2>{});
        if constexpr (KS == 4) {
            __syncthreads();
            exchange(wave ^ C::NW, std::integral_constant<int, 1>{});
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }

    // ---- epilogue: 64 / KS tokens x 128 channels.  Lane (r16, q4) of block (j, i) holds token 16 i + r16 and channels
    // 16 j + 4 q4 + v
    constexpr int KEPT = 4 / KS, ROWS = KS == 4 ? 16 : 32;
    const int m_loc = wm * 64 + (KS == 2 ? 32 * kg : KS == 4 ? 16 * kg : 0);
    const int m_wave = m0 + m_loc, n_wave = n0 + wn * 128;
    if (m_wave >= g.M || n_wave >= g.N) return;
    uint16_t *strip = (uint16_t *)mine;
    const float *sa_w = sc_lds + C::BN + m_loc, *sw_w = sc_lds + wn * 128;
    const bool full = (m_wave + 16 * KEPT <= g.M) && (n_wave + 128 <= g.N) && ((g.ldo & 7) == 0) && (((uintptr_t)g.out & 15) == 0);
#pragma unroll
    for (int r0 = 0; r0 < 16 * KEPT; r0 += ROWS) {
#pragma unroll
        for (int b = 0; b < ROWS / 16; ++b) {
            const float sa = sa_w[r0 + 16 * b + r16];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int nl = 16 * j + 4 * q4;
                const float4 sw = *(const float4 *)(sw_w + nl);
                const v4f &c = acc[j][r0 / 16 + b];
                uint2 hv;
                hv.x = scaled_to_half2(c[0], sa * sw.x, c[1], sa * sw.y);
                hv.y = scaled_to_half2(c[2], sa * sw.z, c[3], sa * sw.w);
                *(uint2 *)(strip + (16 * b + r16) * PITCH + nl) = hv;
            }
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int rr = 0; rr < ROWS; rr += 4) {
            const int row = rr + q4, c8 = 8 * r16;
            const int mo = m_wave + r0 + row, n = n_wave + c8;
            const uint4 q = *(const uint4 *)(strip + row * PITCH + c8);
            uint16_t *dst = g.out + (int64_t)mo * g.ldo + n;
            if (full) {
                const u32x4 qv = {q.x, q.y, q.z, q.w};
                __builtin_nontemporal_store(qv, (u32x4 *)dst);
            } else if (mo < g.M) {
                store_halfs(dst, q, g.N - n);
            }
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

template <int WAVES_M, int WAVES_N, int KS>
hipError_t launch_wide(const GemmArgs &g, const uint32_t *frag, int s_pad, hipStream_t st)
{
    using C = WCfg<WAVES_M, WAVES_N, KS>;
    if (C::SMEM_BYTES > 64 * 1024) {  // said once per device
        static std::atomic<uint64_t> configured{0};
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = 1ull << (dev & 63);
        if (!(configured.load(std::memory_order_relaxed) & bit)) {
            e = hipFuncSetAttribute((const void *)k_gemm_fp4_wide<WAVES_M, WAVES_N, KS>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM_BYTES);
            if (e != hipSuccess) return e;
            configured.fetch_or(bit, std::memory_order_relaxed);
        }
    }
    const int tiles_n = (g.N + C::BN - 1) / C::BN, tiles_m = (g.M + C::BM - 1) / C::BM;
    const int64_t total = (int64_t)tiles_n * tiles_m;
    if (total > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gemm_fp4_wide<WAVES_M, WAVES_N, KS>), dim3((unsigned)total), dim3(C::THREADS),
                       C::SMEM_BYTES, st, g, frag, s_pad, tiles_n, (int)total);
    return hipGetLastError();
}

}  // namespace

// variant: 422 = 128 x 256 tiles of 4 wavefronts; 521 = 128 x 128 of 2 x 2 wavefronts, K split over 2; 611 = 64 x 128
// of 4 wavefronts, K split over 4.  Byte offsets into the packed weights are 32 bits: gemm_fp4_lds_supported.
hipError_t launch_gemm_fp4_wide(const GemmArgs &g, const uint32_t *frag, int variant, hipStream_t st)
{
    if (!gemm_fp4_lds_supported(g)) return hipErrorInvalidValue;
    const int s_pad = fp4_s_pad(g.rw);
    switch (variant) {
    case 422: return launch_wide<2, 2, 1>(g, frag, s_pad, st);
    case 521: return launch_wide<2, 1, 2>(g, frag, s_pad, st);
    case 611: return launch_wide<1, 1, 4>(g, frag, s_pad, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace bwta
