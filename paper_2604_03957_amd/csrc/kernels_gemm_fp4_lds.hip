// BWTA product on the FP4 matrix cores with BOTH operands staged through LDS by direct
// global->LDS loads (global_load_lds_dwordx4: 16 bytes per lane, no register in between).
//
// Why: with the activation fragments loaded straight into registers, each wavefront of a tile
// fetches its own copy of a fragment, and at 2 x 2 blocks of 32 x 32 per wavefront a compute unit
// running its matrix cores flat out would have to pull 64 bytes per clock through its vector memory
// path -- all of that path.  Here a fragment is fetched ONCE per workgroup into LDS and read from
// there by every wavefront that needs it (four of them on the widest tile), and the loads cost no
// VGPR, no LDS store instruction and (addresses being wave-uniform base + lane offset) no
// vector-ALU work.
//
// Layout and roles (Case 1 of the paper's arithmetic rules; operands exact in E2M1, sums exact in
// fp32, see kernels_gemm_fp4.hip):
//   * Workgroup tile (64 WAVES_M) tokens x (32 WN WAVES_N) channels; a wavefront owns 2 x WN blocks
//     of 32 x 32.
//   * K is walked in slabs of 256 (4 MFMA steps).  A slab of activations is 4 fragments of 1 KiB
//     per block of 32 tokens, already in operand order in memory, so one direct load per fragment
//     puts it into LDS exactly as a wavefront reads it back (16 bytes per lane, conflict-free).
//     Weights, 1 bit each, arrive for two slabs at a time: 64 bytes per channel, four neighbouring
//     lanes per channel, so that a load of 16 channels asks the L1 for 16 runs of 64 bytes (with 32
//     channels x 32 bytes per load it was 64 separate 16-byte pieces and the loads alone kept the
//     vector memory path busy for 80 % of the matrix time).  A direct load lays lane l at 16 l, so
//     the lanes of a row fetch its pieces in an order that leaves piece c of row r at slot
//     c ^ (r / 4 % 4): the 8-byte reads of 16 neighbouring rows then meet no bank twice.
//   * Three stages of LDS for the activations, two (of two slabs) for the weights; everything is
//     requested two slabs before it is used.  One workgroup barrier per slab: before it every
//     wavefront waits for ITS OWN requests of that slab (s_waitcnt vmcnt(n): loads complete in order
//     and every wavefront issues the same ones, so n = the younger loads still in flight); after it
//     the slab is visible to all, and what the previous slab was read from is requested again, one
//     load between two MFMA steps.  The last two slabs request nothing.
//     The 64-byte runs and the spread loads together, us on ready fragments whose bits seldom toggle
//     (M x N x K): 2048 x 11008 x 4096 36.4 -> 35.4, 4096 x 4096 x 4096 25.5 -> 25.0, 8192 x 4096 x 1024
//     21.1 -> 20.6; level at 2048 x 4096 x 11008 (34.4 / 34.5), within 1 % at 2048 x 4096 x 4096 and
//     4096 x 3072 x 1024.  With random operands, which the clock pays for, all are level within the noise
//     (40.2 / 40.4 and 38.6 / 38.7 on the first and the fourth).
//   * What bounds it: with all-zero operands the same launch of 2048 x 11008 x 4096 takes 34 us
//     instead of 40 (the clock drops under the power of toggling operands); without direct loads 36.5,
//     without LDS reads 35, without both 31.6.
//   * LDS reads are issued from inline assembly and waited for with explicit lgkmcnt counts: the
//     compiler cannot know which outstanding direct load an LDS read depends on and would otherwise
//     drain all of them (vmcnt(0)) in front of every read, serialising the ring.
//   * Epilogue as in the register-fed kernel (scale bits kept in two registers per thread through
//     the loop), with its LDS scratch in the stages the last slab does not read: the scales
//     are parked there just before the last slab's barrier, the wavefronts' strips follow them, and
//     no wavefront waits for another between its last MFMA and its stores.
#include <type_traits>

#include "bwta_internal.h"
#include "bwta_fp4_tile.h"

namespace bwta {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int WM = 2;  // token blocks of 32 per wavefront

template <int WN, int WAVES_M, int WAVES_N>
struct LCfg {
    static constexpr int BM = 32 * WM * WAVES_M, BN = 32 * WN * WAVES_N;
    static constexpr int NW = WAVES_M * WAVES_N, THREADS = 64 * NW;
    static constexpr int S = 3;                          // activation stages (one slab of 256 k each)
    static constexpr int AF = 4 * (BM / 32);             // activation fragments (1 KiB each) per slab
    static constexpr int WL = BN / 16;                   // weight loads (16 channels, 1 KiB each) per pair of slabs
    static constexpr int A_BYTES = AF * 1024, W_BYTES = WL * 1024;
    static constexpr int W_BASE = S * A_BYTES;           // the two weight stages lie behind the activation stages
    static constexpr int A_ROUNDS = AF / NW, W_ROUNDS = WL / NW;  // direct loads per wavefront: per slab, per pair
    static constexpr int STRIP_BYTES = 32 * (32 * WN + 8) * 2;
    // epilogue scratch: the scales and the first strips in one free activation stage, further strips in
    // the other and in the weight stage the last pair does not use, the rest (if any) behind the ring
    static constexpr int SCALE_BYTES = ((BN + BM) * 4 + 255) / 256 * 256;
    static constexpr int EPI_FIRST = (A_BYTES - SCALE_BYTES) / STRIP_BYTES;
    static constexpr int EPI_SECOND = A_BYTES / STRIP_BYTES;
    static constexpr int EPI_THIRD = W_BYTES / STRIP_BYTES;
    static constexpr int EPI_RING = EPI_FIRST + EPI_SECOND + EPI_THIRD;
    static constexpr int RING_BYTES = W_BASE + 2 * W_BYTES;
    static constexpr int SMEM_BYTES = RING_BYTES + (NW > EPI_RING ? (NW - EPI_RING) * STRIP_BYTES : 0);
    static_assert(AF % NW == 0 && WL % NW == 0, "every wavefront issues the same loads");
    static_assert(BN <= THREADS && BM <= THREADS, "one thread per scale");
    static_assert(SMEM_BYTES <= 160 * 1024, "LDS of one compute unit");
    static_assert(WN == 2 || WN == 4, "read schedules exist for 2 x 2 and 2 x 4 blocks per wavefront");
};

__device__ __forceinline__ void lds_direct_16(const void *src, uint32_t *lds_dst)
{
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src,
                                     (void __attribute__((address_space(3))) *)lds_dst, 16, 0, 0);
}

// one MFMA step of a wavefront: WM token blocks x WN channel blocks
template <int WN>
__device__ __forceinline__ void mfma_step(v16f (&acc)[WN][WM], const u32x4 (&a)[WM], const uint32_t (&w)[WN], uint32_t m88,
                                          uint32_t c22)
{
    v8i vb[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j) {
        vb[j] = widen_w(w[j], m88, c22);
    }
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const v8i va = {(int)a[i].x, (int)a[i].y, (int)a[i].z, (int)a[i].w, 0, 0, 0, 0};
            acc[j][i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vb[j], va, acc[j][i], 4, 4, 0, 0, 0, 0);
        }
}

#define BWTA_LDS_READ_A(dst, off) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(a_addr), "n"(off) : "memory")
#define BWTA_LDS_READ_W(dst, addr, off) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off) : "memory")

// One slab (4 MFMA steps) of a wavefront: its LDS reads, in batches that the 4-bit counter can hold,
// each step waiting only for what it needs (LDS reads return in order), and its MFMAs.
// a_addr: LDS byte address of this lane's first fragment read in the stage; w01 / w23: those of its weight
// words of steps 0, 1 and of steps 2, 3.
// load(t): what the wavefront requests after step t's MFMAs (one load between two steps: a load whose LDS
// address differs from the one before it waits until that one has been consumed).
template <int WN, class Load>
__device__ __forceinline__ void slab_compute(v16f (&acc)[WN][WM], uint32_t a_addr, uint32_t w01, uint32_t w23, uint32_t m88,
                                             uint32_t c22, const Load &load)
{
    u32x2 wlo[WN], whi[WN];
    if constexpr (WN == 4) {
        // 16 reads per slab (8 weight words, 8 fragments), one more than the counter holds: three batches
        u32x4 a0[2], a1[2], a2[2], a3[2];
        BWTA_LDS_READ_W(wlo[0], w01, 0);
        BWTA_LDS_READ_W(wlo[1], w01, 2048);
        BWTA_LDS_READ_W(wlo[2], w01, 4096);
        BWTA_LDS_READ_W(wlo[3], w01, 6144);
        BWTA_LDS_READ_A(a0[0], 0);
        BWTA_LDS_READ_A(a0[1], 4096);
        BWTA_LDS_READ_A(a1[0], 1024);
        BWTA_LDS_READ_A(a1[1], 5120);
        asm volatile("s_waitcnt lgkmcnt(2)"
                     : "+v"(wlo[0]), "+v"(wlo[1]), "+v"(wlo[2]), "+v"(wlo[3]), "+v"(a0[0]), "+v"(a0[1])::"memory");
        {
            const uint32_t w[4] = {wlo[0].x, wlo[1].x, wlo[2].x, wlo[3].x};
            mfma_step<4>(acc, a0, w, m88, c22);
            load(std::integral_constant<int, 0>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        BWTA_LDS_READ_W(whi[0], w23, 0);
        BWTA_LDS_READ_W(whi[1], w23, 2048);
        BWTA_LDS_READ_W(whi[2], w23, 4096);
        BWTA_LDS_READ_W(whi[3], w23, 6144);
        BWTA_LDS_READ_A(a2[0], 2048);
        BWTA_LDS_READ_A(a2[1], 6144);
        asm volatile("s_waitcnt lgkmcnt(6)" : "+v"(a1[0]), "+v"(a1[1])::"memory");
        {
            const uint32_t w[4] = {wlo[0].y, wlo[1].y, wlo[2].y, wlo[3].y};
            mfma_step<4>(acc, a1, w, m88, c22);
            load(std::integral_constant<int, 1>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        BWTA_LDS_READ_A(a3[0], 3072);
        BWTA_LDS_READ_A(a3[1], 7168);
        asm volatile("s_waitcnt lgkmcnt(2)"
                     : "+v"(whi[0]), "+v"(whi[1]), "+v"(whi[2]), "+v"(whi[3]), "+v"(a2[0]), "+v"(a2[1])::"memory");
        {
            const uint32_t w[4] = {whi[0].x, whi[1].x, whi[2].x, whi[3].x};
            mfma_step<4>(acc, a2, w, m88, c22);
            load(std::integral_constant<int, 2>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a3[0]), "+v"(a3[1])::"memory");
        {
            const uint32_t w[4] = {whi[0].y, whi[1].y, whi[2].y, whi[3].y};
            mfma_step<4>(acc, a3, w, m88, c22);
            load(std::integral_constant<int, 3>{});
        }
    } else {
        u32x4 a[4][2];
        // 12 reads in this order; each step waits until its own have returned (reads return in order)
        BWTA_LDS_READ_W(wlo[0], w01, 0);
        BWTA_LDS_READ_W(wlo[1], w01, 2048);
        BWTA_LDS_READ_A(a[0][0], 0);
        BWTA_LDS_READ_A(a[0][1], 4096);
        BWTA_LDS_READ_A(a[1][0], 1024);
        BWTA_LDS_READ_A(a[1][1], 5120);
        BWTA_LDS_READ_W(whi[0], w23, 0);
        BWTA_LDS_READ_W(whi[1], w23, 2048);
        BWTA_LDS_READ_A(a[2][0], 2048);
        BWTA_LDS_READ_A(a[2][1], 6144);
        BWTA_LDS_READ_A(a[3][0], 3072);
        BWTA_LDS_READ_A(a[3][1], 7168);
        // the values pass through the wait so that nothing that uses them can be scheduled above it
        asm volatile("s_waitcnt lgkmcnt(8)" : "+v"(wlo[0]), "+v"(wlo[1]), "+v"(a[0][0]), "+v"(a[0][1])::"memory");
        {
            const uint32_t w[2] = {wlo[0].x, wlo[1].x};
            mfma_step<2>(acc, a[0], w, m88, c22);
            load(std::integral_constant<int, 0>{});
        }
        __builtin_amdgcn_sched_barrier(0);  // keep each step's MFMAs in front of the next wait
        asm volatile("s_waitcnt lgkmcnt(6)" : "+v"(a[1][0]), "+v"(a[1][1])::"memory");
        {
            const uint32_t w[2] = {wlo[0].y, wlo[1].y};
            mfma_step<2>(acc, a[1], w, m88, c22);
            load(std::integral_constant<int, 1>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(2)" : "+v"(whi[0]), "+v"(whi[1]), "+v"(a[2][0]), "+v"(a[2][1])::"memory");
        {
            const uint32_t w[2] = {whi[0].x, whi[1].x};
            mfma_step<2>(acc, a[2], w, m88, c22);
            load(std::integral_constant<int, 2>{});
        }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[3][0]), "+v"(a[3][1])::"memory");
        {
            const uint32_t w[2] = {whi[0].y, whi[1].y};
            mfma_step<2>(acc, a[3], w, m88, c22);
            load(std::integral_constant<int, 3>{});
        }
    }
}

// two workgroups share a compute unit: with eight wavefronts each the register budget is 128, with four 256
template <int WN, int WAVES_M, int WAVES_N, bool WITH_ACC>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) __attribute__((amdgpu_waves_per_eu(WAVES_M * WAVES_N == 8 ? 4 : 2)))
void k_gemm_fp4_lds(GemmArgs g, const uint32_t *__restrict__ frag, int s_pad, int tiles_n, int tiles_total)
{
    using C = LCfg<WN, WAVES_M, WAVES_N>;
    extern __shared__ __attribute__((aligned(1024))) uint32_t smem[];
    int tm, tn;
    tile_of_workgroup(tiles_n, tiles_total, tm, tn);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction: keeps addressing scalar
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int r32 = lane & 31, h = lane >> 5;
    const int m0 = tm * C::BM, n0 = tn * C::BN;
    const int rw = g.rw;
    const int npair = s_pad >> 3;  // pairs of slabs of 4 steps: the fragment buffer is padded to 8 steps

    // ---- scale bits: requested first, kept in registers through the loop
    const bool want_sw = tid < C::BN && n0 + tid < g.N, want_sa = tid < C::BM && m0 + tid < g.M;
    const bool have_sw = want_sw && g.s_w.mode != 0 && g.s_w.ptr != nullptr;
    const bool have_sa = want_sa && g.s_a.mode != 0 && g.s_a.ptr != nullptr;
    const uint16_t *scale_safe = (const uint16_t *)g.wsign;
    const uint16_t sw_bits = *(have_sw ? g.s_w.ptr + (g.s_w.mode == 1 ? 0 : n0 + tid) : scale_safe);
    const uint16_t sa_bits = *(have_sa ? g.s_a.ptr + (g.s_a.mode == 1 ? 0 : m0 + tid) : scale_safe);

    // ---- what this wavefront requests.  Round q of a slab's activation part: fragment f = q NW + wave
    // (token block f / 4, step f % 4).  Round q of a pair's weight part: channels 16 (q NW + wave) .. + 15,
    // 64 bytes each; lane l fetches the 16-byte piece (l % 4) ^ (l / 16) of channel l / 4, so that a quad
    // asks for one run of 64 bytes and piece c of row r lies at slot c ^ (r / 4 % 4) of the row's 64 bytes
    // in LDS.  Sources are a wave-uniform base plus a 32-bit lane offset.
    const char *a_tile = (const char *)frag + (int64_t)tm * (C::BM / 32) * s_pad * 1024;
    const uint32_t a_lane = (uint32_t)lane * 16u;
    // byte offset of this lane's piece of pair 0, round 0 from the weights' base
    const uint32_t w_lane = (uint32_t)(n0 + 16 * wave + (lane >> 2)) * (uint32_t)rw * 4u + 16u * (uint32_t)((lane & 3) ^ (lane >> 4));
    const uint32_t w_last = (uint32_t)g.N * (uint32_t)rw * 4u - 16u;
    auto request_a = [&](int q, int slab, int stage) {
        const int f = q * C::NW + wave;
        const char *src = a_tile + ((int64_t)(f >> 2) * s_pad + 4 * slab + (f & 3)) * 1024;
        lds_direct_16(src + a_lane, smem + stage * (C::A_BYTES / 4) + f * 256);
    };
    auto request_w = [&](int q, int pair) {
        // Past a row's end (K tail) the next row's words arrive, which meet zero activations; channels past
        // the last one are never stored.  Only the matrix's end needs a clamp.
        const uint32_t off = w_lane + (uint32_t)(q * C::NW * 64) * (uint32_t)rw + 64u * (uint32_t)pair;
        lds_direct_16((const char *)g.wsign + (off < w_last ? off : w_last),
                      smem + (C::W_BASE + (pair & 1) * C::W_BYTES) / 4 + (q * C::NW + wave) * 256);
    };

    v16f acc[WN][WM];  // [channel block][token block]
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;

    uint32_t m88 = 0x88888888u, c22 = 0x22222222u;
    asm volatile("" : "+s"(m88));
    asm volatile("" : "+v"(c22));

#pragma unroll
    for (int q = 0; q < C::A_ROUNDS; ++q) request_a(q, 0, 0);
#pragma unroll
    for (int q = 0; q < C::W_ROUNDS; ++q) request_w(q, 0);
#pragma unroll
    for (int q = 0; q < C::A_ROUNDS; ++q) request_a(q, 1, 1);

    // LDS byte addresses of this lane's reads inside a stage.  Row r of a weight stage is its 64 bytes at
    // 64 r; the first slab of a pair reads pieces 0 and 1, the second 2 and 3, at the slots above.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t *)smem;
    const uint32_t a_rd = lds0 + (uint32_t)((wm * WM) * 4096 + lane * 16);  // + i 4096 + step 1024
    const uint32_t w_rd = lds0 + (uint32_t)(C::W_BASE + (wn * WN * 32 + r32) * 64 + ((r32 >> 2) & 3) * 16 + h * 8);  // ^ 16 piece, + j 2048

    // Inside the slab loop a wavefront issues ahead of the wavefronts of the other workgroup on this
    // compute unit that are still setting up or already in their epilogue (scalar address arithmetic,
    // conversions, LDS strips): those fill the gaps.  Measured on the shape that runs several rounds of
    // workgroups per compute unit (2048 x 11008 x 4096): 45.0 -> 43.1 us on the same box; no change on
    // the single-round shapes.
    __builtin_amdgcn_s_setprio(3);
    int stage = 0;
    // One slab: wait for the own requests of it (YOUNGER loads of this wavefront may stay in flight: loads
    // complete in order and every wavefront issues the same ones), then the barrier after which everyone's
    // have landed and everyone is done reading the previous slab.
    auto slab = [&](auto younger, auto half, int pair, auto before_barrier, auto load) {
        __builtin_amdgcn_sched_barrier(0);  // the previous slab's MFMAs stay in front of the wait
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(younger)::value) : "memory");
        before_barrier();
        __builtin_amdgcn_s_barrier();
        const uint32_t a_addr = a_rd + (uint32_t)(stage * C::A_BYTES);
        const uint32_t w = (w_rd + (uint32_t)((pair & 1) * C::W_BYTES)) ^ (32u * decltype(half)::value);
        stage = stage + 1 == C::S ? 0 : stage + 1;
        slab_compute<WN>(acc, a_addr, w, w ^ 16u, m88, c22, load);
    };
    auto nothing = [] {};
    auto no_load = [](auto) {};
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, 1> second{};
    constexpr std::integral_constant<int, C::A_ROUNDS> one_slab{};                     // in flight: a slab's fragments
    constexpr std::integral_constant<int, C::A_ROUNDS + C::W_ROUNDS> slab_and_pair{};  // ... and a pair's weights
    auto two_ahead = [&] { return stage == 0 ? C::S - 1 : stage - 1; };  // the stage the previous slab was read from
    for (int p = 0; p + 1 < npair; ++p) {
        const int st2 = two_ahead();
        slab(one_slab, first, p, nothing, [&](auto t) {
#pragma unroll
            for (int q = decltype(t)::value; q < C::A_ROUNDS + C::W_ROUNDS; q += 4) {
                if (q < C::A_ROUNDS) request_a(q, 2 * p + 2, st2);
                else request_w(q - C::A_ROUNDS, p + 1);
            }
        });
        const int st3 = two_ahead();
        slab(slab_and_pair, second, p, nothing, [&](auto t) {
#pragma unroll
            for (int q = decltype(t)::value; q < C::A_ROUNDS; q += 4) request_a(q, 2 * p + 3, st3);
        });
    }
    // The last pair requests nothing, so the activation stage behind the last slab's and the other weight
    // stage are free before the last slab's barrier, and the stage of the slab before it after that barrier.
    // The first of them takes the scales (written before the barrier, which publishes them); all take the
    // wavefronts' epilogue strips.  So a wavefront goes from its last MFMA into its epilogue without
    // waiting for anyone.
    slab(one_slab, first, npair - 1, nothing, no_load);
    float *sc_lds = nullptr;  // [BN] channel scales, then [BM] token scales
    slab(first, second, npair - 1,
         [&] {
             sc_lds = (float *)(smem + (stage + 1 == C::S ? 0 : stage + 1) * (C::A_BYTES / 4));
             if (tid < C::BN) sc_lds[tid] = have_sw ? half_bits_to_float(sw_bits) : (want_sw ? 1.0f : 0.0f);
             if (tid < C::BM) sc_lds[C::BN + tid] = have_sa ? half_bits_to_float(sa_bits) : (want_sa ? 1.0f : 0.0f);
         },
         no_load);
    __builtin_amdgcn_s_setprio(0);
    // `stage` now names the stage behind the last slab's, where the scales are
    int strip_at;
    if (wave < C::EPI_FIRST) {
        strip_at = stage * C::A_BYTES + C::SCALE_BYTES + wave * C::STRIP_BYTES;
    } else if (wave < C::EPI_FIRST + C::EPI_SECOND) {
        strip_at = (stage + 1 == C::S ? 0 : stage + 1) * C::A_BYTES + (wave - C::EPI_FIRST) * C::STRIP_BYTES;
    } else if (wave < C::EPI_RING) {
        strip_at = C::W_BASE + (npair & 1) * C::W_BYTES + (wave - C::EPI_FIRST - C::EPI_SECOND) * C::STRIP_BYTES;
    } else {
        strip_at = C::RING_BYTES + (wave - C::EPI_RING) * C::STRIP_BYTES;
    }

    const int m_wave = m0 + wm * WM * 32, n_wave = n0 + wn * WN * 32;
    if (WITH_ACC && g.acc) {
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int m = m_wave + 32 * i + r32;
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int n = n_wave + 32 * j + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (m < g.M && n < g.N) g.acc[(int64_t)m * g.N + n] = (int)acc[j][i][v];
                }
        }
    }
    if (!g.out) return;
    uint16_t *strip = (uint16_t *)((char *)smem + strip_at);
    store_tile_fp16<WM, WN>(acc, g, sc_lds + C::BN + wm * WM * 32, sc_lds + wn * WN * 32, strip, m_wave, n_wave, lane);
}

#undef BWTA_LDS_READ_A
#undef BWTA_LDS_READ_W

template <int WN, int WAVES_M, int WAVES_N, bool WITH_ACC>
hipError_t launch_lds(const GemmArgs &g, const uint32_t *frag, int s_pad, hipStream_t st)
{
    using C = LCfg<WN, WAVES_M, WAVES_N>;
    static bool configured = false;  // benign race: setting the attribute twice is harmless
    if (!configured) {
        hipError_t e = hipFuncSetAttribute((const void *)k_gemm_fp4_lds<WN, WAVES_M, WAVES_N, WITH_ACC>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM_BYTES);
        if (e != hipSuccess) return e;
        configured = true;
    }
    if (s_pad < 8) return hipErrorInvalidValue;  // the kernel's tail runs one pair of slabs (the padding gives it)
    const int tiles_n = (g.N + C::BN - 1) / C::BN, tiles_m = (g.M + C::BM - 1) / C::BM;
    const int64_t total = (int64_t)tiles_n * tiles_m;
    if (total > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gemm_fp4_lds<WN, WAVES_M, WAVES_N, WITH_ACC>), dim3((unsigned)total), dim3(C::THREADS),
                       C::SMEM_BYTES, st, g, frag, s_pad, tiles_n, (int)total);
    return hipGetLastError();
}

}  // namespace

// byte offsets into the packed weights, up to a tile of rows and a pair of slabs past their end, are 32 bits
bool gemm_fp4_lds_supported(const GemmArgs &g) { return ((int64_t)g.N + 512) * g.rw * 4 <= 0xffffffffll && g.rw >= 4; }

// The LDS-staged tiled kernel on ready fragments.  variant: 243 = 128 x 256 tiles, 8 wavefronts of
// 64 x 64 (the dispatcher's choice); 223 = 128 x 128 tiles, 4 wavefronts of 64 x 64; 323 = 128 x 256
// tiles, 4 wavefronts of 64 tokens x 128 channels; all with a ring of three slabs.
hipError_t launch_gemm_fp4_lds(const GemmArgs &g, const uint32_t *frag, int variant, hipStream_t st)
{
    const int s_pad = fp4_s_pad(g.rw);
    if (!gemm_fp4_lds_supported(g)) return hipErrorInvalidValue;
#define BWTA_LDS_CASE(ID, WN, WVM, WVN)                                          \
    case ID:                                                                     \
        return g.acc ? launch_lds<WN, WVM, WVN, true>(g, frag, s_pad, st)        \
                     : launch_lds<WN, WVM, WVN, false>(g, frag, s_pad, st);
    switch (variant) {
        BWTA_LDS_CASE(223, 2, 2, 2)
        BWTA_LDS_CASE(243, 2, 2, 4)
        BWTA_LDS_CASE(323, 4, 2, 2)
    default: return hipErrorInvalidValue;
    }
#undef BWTA_LDS_CASE
}

}  // namespace bwta
