// bwta_linear in one launch where it makes at most one round of small workgroups: decode-sized token counts and few
// hundred tokens against narrow matrices.  Such a call is all latency: the launch, two memory round trips, ternarising,
// a chain of MFMAs, the store.  So everything is requested at once and every part is split as far as it goes.
//
//   * A workgroup of eight wavefronts owns 16 tokens (a block of v_mfma_f32_16x16x128_f8f6f4) and 128 / KW channels.
//     All its loads go out before anything is waited for: scales, the strip's activations (all of K up to 6144, 2 NCH
//     groups of 8 per thread), the wavefront's weight words in operand order (four words of a channel per lane and
//     chunk of 512 k: the fragments are made here, so words may be dealt to steps in the order that makes them
//     adjacent).
//   * The strip is ternarised into LDS in operand order (a wavefront takes one word of 16 rows: the 4-byte writes of a
//     quad and its 16 rows are 256 bytes in a row), one barrier, then KW groups of wavefronts share K: the chain of
//     dependent MFMAs and LDS reads is K / (128 KW) steps long.  Their sums meet in LDS in fp32 (whole numbers).
//   * With 32-token strips (k_linear_fused, k_linear_strip) a workgroup ternarises twice as much with half as many
//     wavefronts, and waits for whole slabs in turn.  us replayed, those / this one: 64 x 768 x 768 4.8 / 3.4, 16 x 4096 x
//     1024 5.4 / 3.5, 64 x 4096 x 2048 6.4 / 4.6, 129 x 768 x 4096 9.7 / 6.4, 512 x 768 x 768 4.9 / 3.7.
//   * What bounds it: 1.9 us between empty launches; 0.4 us per 512 k beyond, in which a compute unit takes 16 KB of
//     activations in and ternarises them (31 vector-ALU operations per 8 elements).
#include <atomic>

#include "bwta_internal.h"
#include "bwta_fp4_tile.h"

namespace bwta {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kRowsThreads = 512;

// NCH: chunks of 512 k held (K <= 512 NCH); KW: groups of wavefronts that share K, the other 8 / KW side by side
template <int NCH, int KW>
__global__ __launch_bounds__(kRowsThreads) __attribute__((amdgpu_waves_per_eu(2)))
void k_linear_rows(const uint16_t *__restrict__ A, int64_t lda, GemmArgs g, int strips, int total)
{
    constexpr int NCW = 8 / KW, CPW = (NCH + KW - 1) / KW, PASSES = 2 * NCH, BATCH = PASSES > 24 ? PASSES / 2 : PASSES;
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    float4 *part = (float4 *)(smem + NCH * 1024);  // [8 wavefronts][64 lanes]
    // ids are dealt to the 8 XCDs in turn; an XCD gets neighbouring numbers, strips fastest: the strips of a tile of
    // channels read the same weights
    int strip, tile;
    {
        const int xcd = blockIdx.x & 7, chunk = total >> 3, rem = total & 7;
        const int id = xcd * chunk + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
        tile = id / strips, strip = id - tile * strips;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = wave % NCW, kq = wave / NCW;
    const int r16 = lane & 15, q4 = lane >> 4;
    const int m0 = 16 * strip, n0 = 16 * (NCW * tile + cw), rw = g.rw;

    // ---- requests: scales, this thread's activations (lane j of a quad 8 elements of word 8 p + wave), weight words
    const int row = lane >> 2, j = lane & 3, m = m0 + row, mc = m < g.M ? m : 0;
    const bool have_sa = g.s_a.mode != 0 && g.s_a.ptr != nullptr, have_sw = g.s_w.mode != 0 && g.s_w.ptr != nullptr;
    const uint16_t sa_bits = *(have_sa ? g.s_a.ptr + (g.s_a.mode == 1 ? 0 : mc) : A);
    uint16_t sw_bits[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        int n = n0 + 4 * q4 + v;
        n = n < g.N ? n : g.N - 1;
        sw_bits[v] = *(have_sw ? g.s_w.ptr + (g.s_w.mode == 1 ? 0 : n) : A);
    }
    const uint16_t *a_row = A + (int64_t)mc * lda;
    uint4 x[BATCH];
#pragma unroll
    for (int p = 0; p < BATCH; ++p) x[p] = request_group(a_row, 32 * (8 * p + wave) + 8 * j, g.K);
    // chunk kq + KW i: four words of the lane's channel, one per instruction; words past the row's end meet zeros
    const int n_row = n0 + r16 < g.N ? n0 + r16 : g.N - 1;
    const uint32_t *w_row = g.wsign + (int64_t)n_row * rw;
    uint4 wq[CPW];
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int kw = 16 * (kq + KW * i) + 4 * q4;
        wq[i] = *(const uint4 *)(w_row + (kw < rw ? kw : rw - 4));
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- ternarise the strip into LDS: word q = 16 c + 4 g + e feeds lane group g of step 4 c + e
    const TernaryThr thr = ternary_thresholds(have_sa ? sa_bits : 0x3c00u, m < g.M);
    auto park = [&](int p, const uint4 &xv) {
        const int q = 8 * p + wave;
        uint32_t *dst = smem + ((4 * (q >> 4) + (q & 3)) * 64 + ((q >> 2) & 3) * 16 + row) * 4 + j;
        if (32 * q >= g.K) {  // the whole word lies past the rows' end
            *dst = 0;
            return;
        }
        const uint4 v = 32 * q + 32 > g.K ? finish_group(xv, 32 * q + 8 * j, g.K) : xv;
        *dst = fragment_dword(v, thr, j);
    };
#pragma unroll
    for (int p = 0; p < BATCH; ++p) park(p, x[p]);
    if constexpr (BATCH < PASSES) {
#pragma unroll
        for (int p = 0; p < BATCH; ++p) x[p] = request_group(a_row, 32 * (8 * (BATCH + p) + wave) + 8 * j, g.K);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < BATCH; ++p) park(BATCH + p, x[p]);
    }
    __syncthreads();

    // ---- products
    uint32_t m88 = 0x88888888u, c22 = 0x22222222u;
    asm volatile("" : "+s"(m88));
    asm volatile("" : "+v"(c22));
    const uint4 *a_rd = (const uint4 *)smem + lane;
    v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        const int c = kq + KW * i;
        if (NCH % KW == 0 || c < NCH) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint4 av = a_rd[(4 * c + e) * 64];
                const v8i a = {(int)av.x, (int)av.y, (int)av.z, (int)av.w, 0, 0, 0, 0};
                const v8i w = widen_w(e == 0 ? wq[i].x : e == 1 ? wq[i].y : e == 2 ? wq[i].z : wq[i].w, m88, c22);
                acc[e & 1] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w, a, acc[e & 1], 4, 4, 0, 0, 0, 0);
            }
        }
    }
    v4f sum = acc[0] + acc[1];
    if constexpr (KW > 1) {  // whole numbers: exact in any order
        if (kq) part[wave * 64 + lane] = make_float4(sum[0], sum[1], sum[2], sum[3]);
        __syncthreads();
        if (kq) return;
#pragma unroll
        for (int k = 1; k < KW; ++k) {
            const float4 o = part[(k * NCW + cw) * 64 + lane];
            sum[0] += o.x, sum[1] += o.y, sum[2] += o.z, sum[3] += o.w;
        }
    }

    // ---- lane (r16, q4) holds token r16 and channels 4 q4 .. + 3
    const uint32_t tok_bits = (uint32_t)__shfl((int)sa_bits, 4 * r16);
    const int mo = m0 + r16, n = n0 + 4 * q4;
    if (mo >= g.M || n >= g.N) return;
    const float sa = have_sa ? half_bits_to_float((uint16_t)tok_bits) : 1.0f;
    float f[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) f[v] = sa * (have_sw ? half_bits_to_float(sw_bits[v]) : 1.0f);
    uint2 hv;
    hv.x = scaled_to_half2(sum[0], f[0], sum[1], f[1]);
    hv.y = scaled_to_half2(sum[2], f[2], sum[3], f[3]);
    uint16_t *dst = g.out + (int64_t)mo * g.ldo + n;
    if (n + 4 <= g.N) {
        __builtin_memcpy(dst, &hv, 8);
    } else {
#pragma unroll
        for (int v = 0; v < 3; ++v)
            if (n + v < g.N) dst[v] = (uint16_t)((v < 2 ? hv.x : hv.y) >> (16 * (v & 1)));
    }
}

template <int NCH, int KW>
hipError_t launch_t(const void *A, int64_t lda, const GemmArgs &g, hipStream_t st)
{
    constexpr int SMEM = NCH * 4096 + 8192;
    if (SMEM > 64 * 1024) {  // said once per device
        static std::atomic<uint64_t> configured{0};
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = 1ull << (dev & 63);
        if (!(configured.load(std::memory_order_relaxed) & bit)) {
            e = hipFuncSetAttribute((const void *)k_linear_rows<NCH, KW>, hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
            if (e != hipSuccess) return e;
            configured.fetch_or(bit, std::memory_order_relaxed);
        }
    }
    const int strips = (g.M + 15) / 16, bn = 128 / KW;
    const int64_t total = ((int64_t)g.N + bn - 1) / bn * strips;
    if (total > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_linear_rows<NCH, KW>), dim3((unsigned)total), dim3(kRowsThreads), SMEM, st, (const uint16_t *)A, lda, g, strips,
                       (int)total);
    return hipGetLastError();
}

}  // namespace

// Where it is ahead, by workgroups of 128 channels.  From 3 150 shapes, M 2 .. 1500, N 128 .. 11008, K 64 .. 11008, its time
// over the other route's (replayed):
//   One round (256): 0.62 to 0.81 up to K = 2048, 2 tokens to 1500.  From 129 tokens, against the slab kernel and the tiled
//   product, 0.65 to 0.86 up to 4096, 0.65 to 0.95 at 6000; at 8192 with few of them (up to 64: 0.85; 256: 1.19), at 11008
//   fewer still (32: 0.70; 64: 1.01).  Up to 128 tokens, against ternarise + decode kernel, 0.79 to 0.91 at K = 2560 and
//   3072, level at 4096 and behind from there (5000: 1.2); K = 2049 .. 3072 is left to the two kernels all the same: that
//   bwta_linear takes two launches there is what bwta_linear_launches has promised, and tests hold it to that.
//   Two rounds' worth, which share compute units in pairs: up to K = 1280, to 384 workgroups at 128 tokens (0.79 to 0.98, 1.04 at
//   512), to 512 beyond (0.79 to 0.98; at 640 1.0 to 1.03).
bool linear_rows_supported(const GemmArgs &g)
{
    if (g.M < 2 || g.K < 8 || g.K > 12288 || g.out == nullptr || g.acc != nullptr || fp4_tuning_forced()) return false;
    const int64_t total = ((int64_t)g.M + 15) / 16 * (((int64_t)g.N + 127) / 128);
    if (total > 256) return g.K <= 1280 && total <= (g.M <= 128 ? 384 : 512);
    if (g.M <= 128) return g.K <= 2048;
    return g.K <= 6144 || (g.K <= 8192 && total <= 64) || total <= 32;
}

// groups that share K: as many as leave one round of workgroups and give every group a chunk
static int rows_split(const GemmArgs &g)
{
    const int64_t strips = ((int64_t)g.M + 15) / 16;
    for (int kw = 4; kw > 1; kw /= 2)
        if (strips * (((int64_t)g.N * kw + 127) / 128) <= 256 && g.K > 512 * (kw - 1)) return kw;
    return 1;
}

hipError_t launch_linear_rows(const void *A, int64_t lda, const GemmArgs &g, hipStream_t st)
{
    const int kw = rows_split(g);
#define BWTA_ROWS(N_, K_) \
    if (g.K <= 512 * N_ && kw == K_) return launch_t<N_, K_>(A, lda, g, st);
    BWTA_ROWS(1, 1) BWTA_ROWS(2, 1) BWTA_ROWS(3, 1) BWTA_ROWS(4, 1) BWTA_ROWS(6, 1) BWTA_ROWS(8, 1) BWTA_ROWS(12, 1)
    BWTA_ROWS(2, 2) BWTA_ROWS(3, 2) BWTA_ROWS(4, 2) BWTA_ROWS(6, 2) BWTA_ROWS(8, 2) BWTA_ROWS(12, 2)
    BWTA_ROWS(4, 4) BWTA_ROWS(6, 4) BWTA_ROWS(8, 4) BWTA_ROWS(12, 4) BWTA_ROWS(16, 4) BWTA_ROWS(24, 4)
#undef BWTA_ROWS
    return hipErrorInvalidValue;
}

}  // namespace bwta
