// Internal interface between the host runtime (kl_host.cpp) and the device
// code (kl_device.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include "kl_layout.h"
#include "kl_lds.h"
#include "kl_sync.h"
#include <stddef.h>
#include <stdint.h>

namespace kl {

// Phase selection bits of one launch of the step kernel.
enum : int {
    kPhEmbed = 1, kPhQkv = 2, kPhAttn = 4, kPhOproj = 8, kPhGateUp = 16, kPhDown = 32,
    kPhHead = 64,
    kPhLayer = kPhQkv | kPhAttn | kPhOproj | kPhGateUp | kPhDown,
};

// Everything one step needs, passed by value as the kernel argument.
struct StepParams {
    // shape
    int L, H, nq, nkv, d, F, V, group;
    int Hp, Ap, Fp;            // K extents padded to kTileK: hidden, n_heads*d, ffn
    int qkv_rg;                // row groups of one KV head's q/k/v block
    int o_rg;                  // row groups of the O projection (H / 8)
    int gu_rg;                 // row groups of the gate/up matrix (2 F / 8)
    int down_rg;               // row groups of one FFN column block of the down matrix
    int head_rg;               // row groups of the LM head
    float eps;
    int max_seq;
    // work partition (depends only on nwg and the shape)
    int Sg;                    // workgroups per KV head: w / Sg is the head
    int Sc, Rc, KTc;           // FFN column blocks, workgroups per block, k-tiles per block
    // packed weights
    const uint8_t *arena;      // layer 0 base
    size_t layer_stride;       // bytes between consecutive layers
    size_t off_attn_norm, off_ffn_norm, off_qkv, off_o, off_gu, off_down;
    size_t off_qkv_bias;       // fp32 Q/K/V biases in packed row order (qkv_bias models)
    int qkv_bias;
    // mixture of experts (E > 1): E experts per layer, topk per token; the
    // router (one packed row group) and expert e's gate/up and down matrices
    // at off_gu + e gu_estride, off_down + e down_estride
    int E, topk;
    size_t off_router, gu_estride, down_estride;
    const uint16_t *embed;     // [V][H] bf16, row-major
    const float *final_norm;   // [Hp]
    const uint16_t *lm_head;   // packed tiles
    const float2 *rope;        // [max_seq][d/2] (cos, sin)
    // step arguments
    const int32_t *tokens, *positions;
    // token loop (greedy sampling, one step per launch sequence):
    int pos_add;               // added to every position (step s of a loop: s)
    const unsigned long long *tok_keys;   // non-null: token b is the previous step's argmax
    int32_t *tok_emit;         // non-null: the embedding phase records the tokens it takes
    unsigned long long *amax;  // non-null: the head leaves each sequence's argmax key here
                               // (cleared by the step before)
    unsigned long long *amax_next;   // with amax: the next step's keys, cleared by this step
    int B;
    uint16_t *kc, *vc;         // [L][kv_batch][nkv][cap][d]
    int kv_batch, cap;
    float *logits, *hidden_out;
    // scratch
    long long *xf;             // [max_batch][Hp] residual stream, fixed point (2^-32 units)
    long long *xf2;            // batched path: the other residual buffer (the folds alternate)
    float *xpart;              // batched path: K-slice partials [ks][max_batch][Hp] (O, down)
    int xpart_stride;          // floats between consecutive K-slice partials
    int KSo, KSd;              // K slices of the batched O and down projections
    float *gpart;              // batched path: K-slice partials of the gate/up product
                               // [ks][max_batch][2F rows] and, at other times, of the
                               // q/k/v product [ks][max_batch][nkv * qkv_rg * 8 rows]
    int gpart_stride;          // floats between consecutive gate/up K-slice partials
    int qpart_stride;          // floats between consecutive q/k/v K-slice partials
    int KSg, KSq;              // K slices of the batched gate/up and q/k/v products
    float *ssp;                // batched path: sums of squares of the last RMSNorm step's
                               // rows per kGemmChunkK columns [max_batch][ceil(Hp / chunk)]
    float *q;                  // batched path: [B][nq*d] rotated queries
    // per-sequence path (batch below the model's matrix-core batch): values handed between
    // workgroups as tagged words (value in the low 32 bits, the tag of the
    // writing step and layer in the high 32 bits)
    unsigned *epoch_ptr;       // device word: the current step's first tag (layer l's tag
                               // is *epoch_ptr + l; the step's last phase advances it)
    unsigned *epoch_arrivals;  // device word: workgroups of the step's last phase that have
                               // read it (the last one advances it and clears this)
    unsigned long long *q_ll;  // [B][nq*d] rotated queries (fp32)
    unsigned long long *kv_ll; // [B][nkv][d]: new key (d/2 words: bf16 dims i, i + d/2),
                               // then new value (d/2 words: bf16 dims 2j, 2j + 1)
    unsigned long long *po_ll; // attention parts, [nkv][Sg + B][group][d + 2]: outputs, max
                               // (log2 units) and sum (batched path: [nkv][Sg][..])
    unsigned long long *o_ll;  // [parts of o_heads][B][heads][d] merged attention output (fp32)
    unsigned long long *xa_ll, *xb_ll;   // [B][Hp] residual after the attention, after the
                               // layer (fp32; layer l's input has tag epoch + l)
    unsigned long long *dp_ll; // [B][topk Sc][Hp] down projection's partial sums (fp32)
    int own_max;               // residual rows a workgroup owns, at most (LDS stride)
    unsigned long long *m_ll;  // [B][Fp] SwiGLU output (fp32)
    // batched path: activations as bf16 hi and lo terms (hi + lo ~ the fp32 value)
    uint16_t *act, *act_lo;    // [max_batch][Hp] normalised activations
    uint16_t *actm, *actm_lo;  // [max_batch][Fp] SwiGLU output
    uint16_t *acto, *acto_lo;  // [max_batch][nq*d] attention output
    unsigned long long *bar;   // grid barrier counters (monotonic): group g at [32 (g + 1)]
    unsigned *cnt;             // matrix-core path's local counters: [nkv] q/k/v, then the
                               // RMSNorm slices (256 bytes apart)
    int *err;                  // device error word
    const uint8_t *dummy;      // 16 readable bytes: target of the GEMV ring's spare loads
    int nwg;                   // grid size
    int lds_red, lds_sm, lds_bar;   // dynamic LDS layout (float offsets)
    int batched;               // this step runs the matrix-core path (set by the host)
    int multi;                 // per-sequence path: the B <= kMultiSeq sequences share each
                               // GEMV pass (1), on the matrix cores (2) (set by the host)
    int lds_mm;                // multi = 2: the waves' weight re-layout slots (float offset)
    int o_heads;               // heads that the O projection stages at a time
    unsigned long long *trace; // optional phase timestamps (see kl_set_trace), or null
    int trace_max;             // phases recorded per launch
};

typedef void (*StepKernel)(StepParams, int, int, int);
StepKernel step_kernel_d64(int group);
StepKernel step_kernel_d64_batched(int group);
StepKernel step_kernel_d128(int group);
StepKernel step_kernel_d128_batched(int group);

hipError_t launch_step(const StepParams &p, int first_layer, int last_layer, int phases,
                       bool cooperative, int lds_bytes, hipStream_t stream);
// Adds the same launch as a kernel node of graph g after 'dep' (null: none);
// cooperative nodes carry the graph's cooperative attribute.
hipError_t add_step_node(hipGraph_t g, hipGraphNode_t *node, const hipGraphNode_t *dep,
                         const StepParams &p, int first_layer, int last_layer, int phases,
                         bool cooperative, int lds_bytes);
hipError_t step_kernel_setup(int d, int group, int lds_bytes, int *max_blocks_per_cu);

// The static scratch of kl_decode_step_noalloc: one array per device, of
// this many bytes, held until the process ends.
constexpr size_t kStaticScratchBytes = size_t(32) << 20;
// It is followed by a reserve for the larger hand-offs as tagged words: up to
// 7 sequences' down partials in 64 column blocks (experts), 20K rows wide.
constexpr size_t kStaticWordBytes = size_t(88) << 20;
// This device's address of the static scratch ('device' must be current);
// resolved with hipGetSymbolAddress once per device, then cached.
hipError_t static_scratch_address(int device, uint8_t **out);
// Zero 'bytes' (a multiple of 16, 16-byte aligned) at p with a fill kernel.
hipError_t launch_zero(void *p, size_t bytes, hipStream_t stream);
hipError_t launch_read_stream(const void *p, size_t bytes, int workgroups, uint32_t *out,
                              hipStream_t stream);

// tokens[b] = the token of argmax key keys[b] (-1 where there is none), b < n; then
// clear[b] = 0 (the keys of the next loop's first step; may be 'keys').
hipError_t launch_emit_tokens(int32_t *tokens, const unsigned long long *keys,
                              unsigned long long *clear, int n, hipStream_t stream);

hipError_t launch_pack_rows(uint16_t *dst, int n_rg, int kt, int K, int ld, const int32_t *rowmap,
                            const uint16_t *src0, const uint16_t *src1, const uint16_t *src2,
                            hipStream_t stream);
// dst[r] = fp32 bias of packed q/k/v row r (rowmap as for the matrix; the
// sources bq, bk, bv are source ids 0, 1, 2).
hipError_t launch_pack_bias(float *dst, int rows, const int32_t *rowmap, const uint16_t *bq,
                            const uint16_t *bk, const uint16_t *bv, hipStream_t stream);
hipError_t launch_gain_to_f32(float *dst, const uint16_t *src, int n, int npad,
                              hipStream_t stream);

}  // namespace kl
