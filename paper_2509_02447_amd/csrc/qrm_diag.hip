// Diagnostic entry points (include/qrm_diag.h): flags for A/B runs and a probe of the matrix pipes.  Bench and
// test tooling; nothing of the detection path lives here.
#include <math.h>

#include <vector>

#include "qrm_ctx.h"
#include "../../include/qrm_diag.h"

using namespace qrm;

namespace qrm {
namespace {

// What the matrix pipes sustain with nothing else going on.  Eight wavefronts per CU issue
// v_mfma_f32_32x32x16_bf16 back to back on four operand sets taken from `src` (8192 floats: 4096 for the A
// side, 4096 for the B side).  The clock of the part follows its power budget, and the power of a matrix
// instruction follows the data: zeros run at the published rate, random data do not.
__global__ __launch_bounds__(512) void matrix_rate_kernel(const float *__restrict__ src, int iters, float *__restrict__ out)
{
    bf16x8 a[4], b[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            a[s][i] = (bf16_t)src[((s * 8 + i) * 512 + threadIdx.x) % 4096];
            b[s][i] = (bf16_t)src[((s * 8 + i) * 512 + threadIdx.x) % 4096 + 4096];
        }
    f32x16 acc[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[s][i] = 0.f;
#pragma unroll 1
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], b[s], acc[s], 0, 0, 0);
    }
    out[blockIdx.x * 512 + threadIdx.x] = acc[0][0] + acc[1][1] + acc[2][2] + acc[3][3];
}

hipError_t launch_matrix_rate(const float *src, int iters, int blocks, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(matrix_rate_kernel, dim3(blocks), dim3(512), 0, s, src, iters, out);
    return hipGetLastError();
}

} // namespace
} // namespace qrm

extern "C" {

qrm_status qrm_diag_set_flags(qrm_ctx *c, int32_t flags)
{
    if (!c) return QRM_E_INVALID;
    if (flags & ~(QRM_DIAG_NO_FUSED_PAIRS | QRM_DIAG_POISON_WORKSPACE | QRM_DIAG_FUSE_ALWAYS | QRM_DIAG_CHAIN_ALWAYS | QRM_DIAG_NO_CHAIN | 0xFF00)) return fail(c, QRM_E_INVALID, "unknown diagnostic flag");
    c->diag_flags = flags;
    return QRM_OK;
}

qrm_status qrm_diag_chain_patience(qrm_ctx *c, int32_t looks)
{
    if (!c) return QRM_E_INVALID;
    c->chain_patience = looks;
    return QRM_OK;
}

// The state that launches on `stream` (or qrm_detect_static's) keep, or null.
static ChainMemory *chain_memory(qrm_ctx *c, void *stream, int shared)
{
    if (shared) return static_chain_memory(c->device);
    for (QrmSlot &sl : c->slots)
        if (sl.used && sl.stream == (hipStream_t)stream && sl.chain.words) return &sl.chain;
    return nullptr;
}

qrm_status qrm_diag_chain_count(qrm_ctx *c, void *stream, int32_t shared, int32_t image, uint32_t value)
{
    if (!c) return QRM_E_INVALID;
    ChainMemory *m = chain_memory(c, stream, shared);
    if (!m || image < 0 || image >= kChainCounters) return fail(c, QRM_E_INVALID, "no such workspace or image");
    hipError_t e = hipSetDevice(c->device);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(chain_counter(m->words, image), &value, sizeof value, hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(c, e, "hipMemcpy(chain state)");
    return QRM_OK;
}

qrm_status qrm_diag_chain_left_over(qrm_ctx *c, void *stream, int32_t shared, uint32_t value)
{
    if (!c) return QRM_E_INVALID;
    ChainMemory *m = chain_memory(c, stream, shared);
    if (!m) return fail(c, QRM_E_INVALID, "no such workspace");
    const std::vector<uint32_t> words(kChainStateBytes / 4, value);
    hipError_t e = hipSetDevice(c->device);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(m->words, words.data(), kChainStateBytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(c, e, "hipMemcpy(chain state)");
    m->dirty = true;
    return QRM_OK;
}

qrm_status qrm_diag_chain_rule(int32_t channels, int32_t blocks, int32_t n_img, int32_t h, int32_t w, int32_t num_cu, int32_t *fits,
                               int32_t *taken)
{
    if ((channels != 32 && channels != 64) || blocks < 1 || n_img < 1 || h < 1 || w < 1 || num_cu < 1 || !fits || !taken) return QRM_E_INVALID;
    const ConvGeom g{n_img, h, w, (h + kRows - 1) / kRows, (w + kTileW - 1) / kTileW};
    const ChainPlan p = conv_chain_plan(g, channels, blocks, num_cu);
    *fits = p.fits;
    *taken = p.fits && conv_chain_faster(g, channels, p, blocks, num_cu);
    return QRM_OK;
}

qrm_status qrm_diag_matrix_rate(qrm_ctx *c, int32_t data, double *tflops)
{
    if (!c) return QRM_E_INVALID;
    if (data < 0 || data > 2 || !tflops) return fail(c, QRM_E_INVALID, "data is 0 (zeros), 1 (a constant) or 2 (random); tflops must not be NULL");
    hipError_t e = hipSetDevice(c->device);
    if (e != hipSuccess) return hip_fail(c, e, "hipSetDevice");
    // operands: A side like rounded weights (normal, small), B side like activations after a ReLU
    std::vector<float> h(8192);
    uint64_t state = 0x9E3779B97F4A7C15ull;
    auto uni = [&]() {
        state = state * 6364136223846793005ull + 1442695040888963407ull;
        return ((double)(state >> 11) + 1.0) / 9007199254740994.0;
    };
    for (int i = 0; i < 8192; ++i) {
        const double n = sqrt(-2.0 * log(uni())) * cos(6.283185307179586 * uni());
        h[i] = data == 0 ? 0.f : data == 1 ? 1.5f : (float)(i >= 4096 ? (n > 0 ? n : 0.0) : 0.06 * n);
    }
    const int blocks = c->num_cu, iters = 8000, reps = 3;
    float *d_src = nullptr, *d_out = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    e = hipMalloc((void **)&d_src, h.size() * 4);
    if (e == hipSuccess) e = hipMalloc((void **)&d_out, (size_t)blocks * 512 * 4);
    if (e == hipSuccess) e = hipMemcpy(d_src, h.data(), h.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) e = launch_matrix_rate(d_src, iters, blocks, d_out, nullptr); // warm-up
    if (e == hipSuccess) e = hipEventRecord(e0, nullptr);
    for (int r = 0; r < reps && e == hipSuccess; ++r) e = launch_matrix_rate(d_src, iters, blocks, d_out, nullptr);
    if (e == hipSuccess) e = hipEventRecord(e1, nullptr);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (d_src) (void)hipFree(d_src);
    if (d_out) (void)hipFree(d_out);
    if (e != hipSuccess) return hip_fail(c, e, "matrix rate probe");
    const double flops = (double)reps * blocks * 8 * (double)iters * 4 * 32768.0; // 2 * 32 * 32 * 16 per instruction
    *tflops = flops / ((double)ms * 1e-3) / 1e12;
    return QRM_OK;
}

qrm_status qrm_diag_pair_split(int32_t n_img, int32_t h, int32_t w, int32_t last, int32_t num_cu, int32_t *part, int32_t *per,
                               int32_t *cost)
{
    if (n_img < 1 || h < 1 || w < 1 || num_cu < 1 || !part || !per || !cost) return QRM_E_INVALID;
    const ConvGeom g{n_img, h, w, (h + kRows - 1) / kRows, (w + kTileW - 1) / kTileW};
    const PairSplit p = conv_pair_split(g, last != 0, num_cu);
    *part = p.part;
    *per = p.per;
    *cost = p.cost;
    return QRM_OK;
}

qrm_status qrm_diag_wide_schedule(int32_t n_img, int32_t h, int32_t w, int32_t num_cu, int32_t *fused, double *single_us,
                                  double *fused_us)
{
    if (n_img < 1 || h < 1 || w <= kTileW || num_cu < 1 || !fused || !single_us || !fused_us) return QRM_E_INVALID;
    const ConvGeom g{n_img, h, w, (h + kRows - 1) / kRows, (w + kTileW - 1) / kTileW};
    const WideCost c = conv_wide_cost(g, num_cu);
    *fused = wide_tiles_fused(g, num_cu);
    *single_us = c.single_us;
    *fused_us = c.fused_us;
    return QRM_OK;
}

qrm_status qrm_diag_last_lines(int32_t n_img, int32_t h, int32_t w, int32_t n_blocks, int32_t num_cu, int32_t *row_pairs,
                               int64_t *bytes)
{
    if (n_img < 1 || h < 1 || w < 1 || n_blocks < 2 || num_cu < 1 || !row_pairs || !bytes) return QRM_E_INVALID;
    const ConvGeom g{n_img, h, w, (h + kRows - 1) / kRows, (w + kTileW - 1) / kTileW};
    qrm_ctx c;
    c.num_cu = num_cu;
    c.has_ext = c.collapse = c.pairable = true;
    c.n_blocks = n_blocks;
    c.C = 64;
    *row_pairs = conv_pair_last_sums(g, num_cu).pairs ? 1 : 4;
    *bytes = (int64_t)ws_layout(&c, n_img, h, w, false).total;
    return QRM_OK;
}

qrm_status qrm_diag_host_plan(int32_t channels, int32_t n_blocks, int32_t H, int32_t W, int32_t tile, int32_t chunk_images,
                              int32_t used, int32_t num_cu, int32_t *first, int32_t *rest, int32_t *lent)
{
    if ((channels != 32 && channels != 64) || n_blocks < 1 || tile < 1 || tile > H || tile > W || chunk_images < 1 || used < 1 ||
        num_cu < 1 || !first || !rest || !lent)
        return QRM_E_INVALID;
    const HostPlan p = plan_host_upload(channels, n_blocks, 0, H, W, tile, chunk_images, used, num_cu);
    *first = p.first;
    *rest = p.rest;
    *lent = p.lent_cu;
    return QRM_OK;
}

qrm_status qrm_diag_preprocess_strips(int64_t N, int32_t T, int32_t *strips)
{
    if (N < 1 || T < 1 || !strips) return QRM_E_INVALID;
    *strips = preprocess_strips(N, T, T % 4 == 0);
    return QRM_OK;
}

qrm_status qrm_diag_rs_lanes(int32_t n, int32_t k, int64_t N, int32_t *lanes)
{
    if (k < 1 || n <= k || n > 255 || N < 1 || !lanes) return QRM_E_INVALID;
    RsParams p{};
    p.n = n;
    p.k = k;
    p.two_t = n - k;
    *lanes = rs_lanes_per_word(p, N);
    return QRM_OK;
}

} // extern "C"
