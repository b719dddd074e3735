// Internal declarations shared by the HIP sources of libqrm (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "../../include/qrm.h"

namespace qrm {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 4;     // output rows per strip of the conv kernels
constexpr int kTileW = 64;   // output columns per strip
constexpr int kHaloW = kTileW + 2;

// First layer: K = 9 taps x 4 channels in 16-wide k chunks of two taps for either half of a wavefront.  Tap (3 dy + dx) that
// half `half` reads as its tap j of chunk q.  dy is the same for both halves where it can be: the kernels then find an operand's
// row without vector instructions.
constexpr int kFirstFrags = 5; // chunks 0 .. 2 with the weights' bf16 high parts, chunks 0, 1 with the residuals; tap 8's residual is chunk 2's second tap
__host__ __device__ constexpr int first_tap(int q, int half, int j)
{
    return q == 0 ? 3 * j + half : q == 1 ? (j == 0 ? 6 + half : 3 * half + 2) : 8;
}

// Geometry of one extractor pass over a micro-batch.
struct ConvGeom {
    int n_img;      // images in this launch
    int h, w;       // tile height / width (conv domain)
    int strips;     // ceil(h / kRows)
    int colblks;    // ceil(w / kTileW)
};

// Source of the first convolution: raw u8 planes of the whole image plus tile origin.
struct TileSrc {
    const uint8_t *img; // [N,3,H,W]
    const int32_t *off; // [N,2] (y,x) or nullptr
    int H, W;
    float mean[3], inv_std[3];
};

// ---- launchers (each enqueues on `s`, returns hipGetLastError()) ----------

hipError_t launch_extract_tiles(const uint8_t *img, int64_t N, int H, int W, const int32_t *off, int tile,
                                uint8_t *out, hipStream_t s);

// The same crops out of images in page-locked host memory the device can read (img: its device address), on `workgroups`
// compute units.
hipError_t launch_gather_host_tiles(const uint8_t *img, int64_t N, int H, int W, const int32_t *off, int tile, uint8_t *out,
                                    int workgroups, hipStream_t s);
// Which chunks of a streamed pass come as tiles that way and which as whole images: the first one (nothing runs beside its
// upload), the rest; on how many compute units, and how many of those the kernels that run beside it leave free.
// final_slices: groups of 64 output channels of a final convolution that runs per pixel; used: staging buffers in use.
struct HostPlan {
    bool first, rest;
    int first_workgroups, rest_workgroups, lent_cu;
};
HostPlan plan_host_upload(int C, int n_blocks, int final_slices, int H, int W, int tile, int chunk_images, int used, int num_cu);

// How the tiles of a launch are dealt to workgroups (see make_partition).
struct Partition {
    int per;    // tiles per workgroup
    int blocks; // grid size
};
Partition make_partition(int64_t n_img, int tiles_per_image, int target_blocks);

// Sampled per-image channel sums of a launch's output, as its consumer reads them.
struct MeanIn {
    const float *rec; // [n_img][recs][C], or null: none
    int recs;         // records per image
    float inv_cnt;    // 1 / pixels of an image behind its records
};
// What the last block leaves of an image for the head: `lines` lines of C sums.  Lines 0 .. first_col-1: the whole tile, a
// line per piece of its rows, column block and block of 32 columns; from first_col / last_col on: the first / last column, a
// line per piece; from rows on: the first, then the last row, a line per column block and block of 32 columns; from corners
// on: top left, top right, bottom left, bottom right.  A piece is kChunk row pairs in the fused kernel, the rows one
// wavefront finishes at a time in the single-block one.  seam: the last column was computed apart and is missing from the
// whole-tile and the row lines.
struct LastSums {
    int lines, first_col, last_col, rows, corners, seam;
    int pairs; // not 0: a piece is one row pair, and there are this many of them
    int64_t stride; // 16-byte pieces from an image's lines to the next one's; 0: they follow each other
};
MeanIn conv_first_samples(const ConvGeom &g, int C); // (rec null)
MeanIn conv_mid_samples(const ConvGeom &g, int C);
MeanIn conv_pair_samples(const ConvGeom &g);

// conv1: crop + normalise + conv3x3 (3 -> C, bf16 high + residual weights) + bias + ReLU -> bf16 NHWC;
// tout (optional): sampled channel sums of the output, conv_first_samples() says how many
hipError_t launch_conv_first(const TileSrc &src, const ConvGeom &g, int C, const bf16_t *wfrag, const float *bias,
                             float *tout, const Partition &part, bf16_t *out, hipStream_t s);

// conv3x3 C -> C + bias + ReLU, bf16 NHWC in/out.  Offsets inside an image are 32-bit.
// tin / rsum: channel sums of the input and the summed weight-rounding residual [c_in][c_out] used to correct the
// bias (tin.rec and rsum may be null).  tout: channel sums of the output (conv_mid_samples()).  last: no activations
// are written, tout receives lines of channel sums (conv_mid_last_sums()).
LastSums conv_mid_last_sums(const ConvGeom &g, int C);
hipError_t launch_conv_mid(const uint8_t *in, const ConvGeom &g, int C, const bf16_t *wfrag,
                           const float *bias, const MeanIn &tin, const float *rsum, float *tout,
                           const Partition &part, bool last, bf16_t *out, hipStream_t s);

// Two consecutive blocks in one launch, the activations between them staying in LDS (C = 64:
// conv_pair_supported; tiles wider than 64 columns are walked through in column blocks and need `seam`,
// conv_pair_seam_bytes() bytes of scratch).  in: the input activations.
// first != nullptr: the first of the two is the network's first block (raw u8 tiles, wfrag_a / bias_a of that
// block; in / tin / rsum_a unused); otherwise both are C -> C blocks and tin / rsum_a are as for
// launch_conv_mid (first block only: the second block's weights are rounded so that it needs no correction).
// tout: channel sums of the output (conv_pair_samples()).  last: the second block is the network's last one: no
// activations are written, tout receives lines of channel sums (conv_pair_last_sums()).
bool conv_pair_supported(int C, const ConvGeom &g);
// How the row pairs of a launch are dealt to workgroups.
struct PairSplit {
    bool part;      // runs that begin and end inside images; otherwise whole images
    int per;        // pieces (kChunk row pairs each with `last`, one otherwise) per workgroup
    int workgroups;
    int cost;       // of the longest workgroup (pair_cost)
};
struct WideCost {
    double single_us, fused_us; // estimates for eight blocks
};
WideCost conv_wide_cost(const ConvGeom &g, int num_cu);
// Whether tiles wider than one column block run the fused schedule.
bool wide_tiles_fused(const ConvGeom &g, int num_cu);
PairSplit conv_pair_split(const ConvGeom &g, bool last, int num_cu);
LastSums conv_pair_last_sums(const ConvGeom &g, int num_cu);
size_t conv_pair_seam_bytes(const ConvGeom &g, int num_cu);
hipError_t launch_conv_pair(const uint8_t *in, const TileSrc *first, const ConvGeom &g, int C,
                            const bf16_t *wfrag_a, const bf16_t *wfrag_b, const float *bias_a, const float *bias_b,
                            const MeanIn &tin, const float *rsum_a, float *tout, bool last, int num_cu,
                            uint8_t *seam, bf16_t *out, hipStream_t s);

// All blocks of a batch of few tiles in one launch.
struct ChainPlan {
    bool fits;           // the launch takes such a batch
    bool one_round;      // with an item per compute unit at most
    int rows;            // of an item
    int chunk;           // images that an XCD takes at a time
    int64_t items;       // of a block of a chunk
};
// Images times blocks of a launch: 128 bytes each, 256 KB for each of a context's nine workspaces.  Larger batches take the other ways
// (512 images of four blocks fit, 409 of five, 256 of eight).
constexpr int kChainCounters = 2048;
constexpr size_t kChainStateBytes = (size_t)(9 * 32 + kChainCounters * 32) * 4; // what a launch keeps beside the workspace
// That memory when the launch behind conv_chain's is to clear it (words null: it is not), and what the launch was about.
struct ChainState {
    uint32_t *words;
    uint32_t *lost;              // set where items are missing (null: nobody is told)
    int blocks, n_img;
    uint32_t first_items, items; // of an image, in the first block and in another one
};
uint32_t *chain_counter(uint32_t *words, int image); // items that the first block has done of it
ChainState conv_chain_state(uint32_t *words, uint32_t *lost, const ConvGeom &g, const ChainPlan &p, int blocks);
ChainPlan conv_chain_plan(const ConvGeom &g, int C, int blocks, int num_cu);
bool conv_chain_faster(const ConvGeom &g, int C, const ChainPlan &p, int blocks, int num_cu);
LastSums conv_chain_last_sums(const ConvGeom &g, int C);
// blocks: of the network, from the first on; block b writes act[b & 1] and sampled channel sums to rec[b & 1] (conv_first_samples(),
// then those of conv_mid_samples()).  lines not null: the
// last of them leaves lines of sums there, an image's in the place of its activations (conv_chain_last_sums()).  state: all zeros;
// the launch behind this one clears it.  patience: looks that a wait takes before it gives up (below zero: the usual number).
hipError_t launch_conv_chain(const TileSrc &src, const ConvGeom &g, int C, const ChainPlan &p, int blocks, const bf16_t *w_first,
                             const bf16_t *w_mid, const float *bias, const float *rsum, uint8_t *act0, uint8_t *act1, float *rec0,
                             float *rec1, float *lines, uint32_t *state, int patience, int num_cu, hipStream_t s);
hipError_t launch_clear_chain(uint32_t *state, hipStream_t s);

struct RsParams {
    int m, q, n, k, two_t, fcr;
    const uint8_t *tab; // device, the table image of the code (rs_table_image), 16-byte aligned
    int tab_bytes;      // what a launch takes of it into LDS, a multiple of 16
    int tab2_bytes;     // of the second image behind it, if there is one
};

// Key verification: `key` device [k] symbols; matches null = no verification.
struct KeyArgs {
    const uint8_t *key = nullptr;
    int tau = 0;
    int32_t *matches = nullptr; // [N] number of message bits equal to the key's
    uint8_t *detected = nullptr; // [N] matches >= tau, or null
};

// The word of an image, decoded where its bits are made (rs.tab null: not there).  Pointers: the first image's.
struct WordArgs {
    RsParams rs{};
    uint8_t *msg = nullptr, *cw = nullptr; // cw may be null
    int8_t *nerr = nullptr;
    KeyArgs key{};
};
bool head_decodes(const RsParams &p, int64_t N); // whether the head of N images is to do that

// recs / sums: channel sums of the last block -> final conv + average pool in closed form -> linear -> logits,
// bits, symbols, decoded words.  wft: final conv weights fp32, [C*9][nbp] (k = c*9 + tap major)
hipError_t launch_head(const float *recs, const LastSums &sums, int C, int64_t n_img, int n_bits, int nbp, float inv_hw,
                       const float *wft, const float *fbias, const float *lin_w, const float *lin_b, float *logits,
                       uint8_t *bits, uint8_t *symbols, int m, const WordArgs &word, const ChainState &chain, hipStream_t s);

// final conv3x3 C -> nbp (n_bits padded to 64s) (+bias, optional ReLU) + sum over pixels -> partial sums
// partial: f32 [n_img][conv_final_lines()][nbp], each line over a part of the image that does not depend on `part`
// (conv_final_partition())
int conv_final_lines(const ConvGeom &g);
Partition conv_final_partition(int64_t n_img, int tiles_per_image, int num_cu, int C, int nbp);
hipError_t launch_conv_final(const uint8_t *in, const ConvGeom &g, int C, int nbp, const bf16_t *wfrag,
                             const float *bias, int relu, float *partial, const Partition &part, hipStream_t s);

// pooled = sum(partials)/(h*w); logits = lin_w * pooled + lin_b; bits; symbols (MSB first, m bits each)
// fbias: optional bias of the final convolution, added to the pooled value
hipError_t launch_linear_pack(const float *partial, int lines, int nbp, int64_t n_img, int n_bits, float inv_hw,
                              const float *fbias, const float *lin_w, const float *lin_b, float *logits, uint8_t *bits,
                              uint8_t *symbols, int m, const ChainState &chain, hipStream_t s);

// bf16 NHWC -> f32 NCHW (diagnostic)
hipError_t launch_nhwc_to_nchw(const bf16_t *in, int64_t n_img, int h, int w, int C, float *out, const ChainState &chain, hipStream_t s);

// The tables the decoding kernels keep in LDS for this code, laid out once per context (p.tab unused; sets p.tab_bytes; codes
// with two ways of dealing a word to lanes have an image for either, one behind the other);
// exp2: alpha^0 .. alpha^(2 ord - 1), lg: logarithms of 1 .. q - 1
std::vector<uint8_t> rs_table_image(RsParams &p, const std::vector<uint8_t> &exp2, const std::vector<uint8_t> &lg);
int rs_lanes_per_word(const RsParams &p, int64_t N); // of a launch of N words
hipError_t launch_rs_decode(const RsParams &p, const uint8_t *sym, int64_t N, uint8_t *msg, uint8_t *cw, int8_t *nerr,
                            const KeyArgs &key, hipStream_t s);
// matches / detected for messages already in memory (msg device [N,k])
hipError_t launch_verify(const RsParams &p, const uint8_t *msg, int64_t N, const KeyArgs &key, hipStream_t s);

// Variance-based tile selection: origin of the first window with the largest weighted sum of channel variances.
// off_yx device [N,2]; scores device [N, nH*nW] or null; w: channel weights.
bool select_tiles_supported(int H, int W, int win, int stride);
hipError_t launch_select_tiles_variance(const uint8_t *img, int64_t N, int H, int W, int win, int stride,
                                        const double w[3], int32_t *off_yx, double *scores, hipStream_t s);

// Fused pre-processing: raw u8 [N,H_in,W_in,3] -> resize (shorter side x) -> centre crop x -> planar u8
// [N,3,T,T], the whole crop (T = x) or a tile of it at off (device [N,2] or null).
bool preprocess_supported(int H_in, int W_in, int x, int T);
int preprocess_strips(int64_t N, int T, bool vec); // workgroups per image; vec: T and the output are multiples of 4
hipError_t launch_preprocess(const uint8_t *raw, int64_t N, int H_in, int W_in, int x, const int32_t *off, int T,
                             uint8_t *out, hipStream_t s);

// host-side helpers
uint16_t f32_to_bf16_rne(float f);

} // namespace qrm
