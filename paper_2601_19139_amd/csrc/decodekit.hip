// Host side of the decode-step library: handles, argument checks, block
// accounting, workspace carving and kernel launches.  See include/decodekit.h
// for the contract of every entry point.
#include "../../include/decodekit.h"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <set>
#include <vector>

#include "dk_attention.hip.h"
#include "dk_attention_mfma.hip.h"
#include "dk_attention_prefill.hip.h"
#include "dk_fused.hip.h"
#include "dk_gemm.hip.h"
#include "dk_gemm_shared.hip.h"
#include "dk_gemm_plan.h"
#include "dk_gemv.hip.h"
#include "dk_moe.hip.h"
#include "dk_sample.hip.h"

#include <mutex>

// Device scratch of dk_decode_step_static: one copy per GPU, held until the process ends.  In host
// code this name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[DK_STATIC_SCRATCH_BYTES];

namespace {

thread_local char g_err[512] = "";

// Per GPU: the address of that GPU's copy of `scratch` (looked up on the entry point's first call
// there) and the model whose step used it last (the persistent kernel keeps state in it).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};
const void *g_scratch_owner[kMaxDevices] = {};

dk_status fail(dk_status code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

#define DK_HIP(expr)                                                                        \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(DK_E_HIP, "%s: %s", #expr, hipGetErrorString(e_));                  \
    } while (0)

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Per-kernel timing of a profiled step: every launch carries a start and a stop
// event (the dispatch's own timestamps, not the gaps between launches).
struct Profiler {
    struct Pending { int cls; hipEvent_t e0, e1; };
    std::vector<hipEvent_t> free_events;
    std::vector<Pending> pending;
    double ms[DK_K_COUNT] = {};
    int64_t launches[DK_K_COUNT] = {};
    bool take(int cls, hipEvent_t *e0, hipEvent_t *e1)
    {
        hipEvent_t ev[2];
        for (auto &e : ev) {
            if (!free_events.empty()) { e = free_events.back(); free_events.pop_back(); }
            else if (hipEventCreate(&e) != hipSuccess) return false;
        }
        *e0 = ev[0];
        *e1 = ev[1];
        pending.push_back({cls, ev[0], ev[1]});
        return true;
    }
    ~Profiler()
    {
        for (auto &p : pending) { (void)hipEventDestroy(p.e0); (void)hipEventDestroy(p.e1); }
        for (auto e : free_events) (void)hipEventDestroy(e);
    }
};
thread_local Profiler *g_prof = nullptr;   // set for the duration of a profiled step

// Launch through here so that a profiled step can time each kernel.
#define DK_LAUNCH(cls, kernel, grid, block, lds, st, ...)                                      \
    do {                                                                                       \
        hipEvent_t e0_, e1_;                                                                   \
        if (g_prof != nullptr && g_prof->take(cls, &e0_, &e1_))                                \
            hipExtLaunchKernelGGL(kernel, grid, block, lds, st, e0_, e1_, 0, __VA_ARGS__);     \
        else                                                                                   \
            hipLaunchKernelGGL(kernel, grid, block, lds, st, __VA_ARGS__);                     \
    } while (0)

dk_status check_config(const dk_model_config *c)
{
    if (!c) return fail(DK_E_INVALID_ARG, "config is NULL");
    if (c->n_layers <= 0 || c->hidden <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 ||
        c->vocab <= 0)
        return fail(DK_E_INVALID_ARG, "config has a non-positive dimension");
    if (c->head_dim != 64 && c->head_dim != 128)
        return fail(DK_E_UNSUPPORTED_SHAPE, "head_dim %d (64 or 128 supported)", c->head_dim);
    if (c->n_q_heads % c->n_kv_heads)
        return fail(DK_E_UNSUPPORTED_SHAPE, "n_q_heads %d is not a multiple of n_kv_heads %d",
                    c->n_q_heads, c->n_kv_heads);
    const int G = c->n_q_heads / c->n_kv_heads;
    if (G < 1 || G > 8)
        return fail(DK_E_UNSUPPORTED_SHAPE, "query group size %d (1..8 supported)", G);
    if (c->hidden % 8) return fail(DK_E_UNSUPPORTED_SHAPE, "hidden %d not a multiple of 8", c->hidden);
    if (c->n_experts < 0 || c->n_experts > DK_MAX_EXPERTS)
        return fail(DK_E_UNSUPPORTED_SHAPE, "n_experts %d (at most %d)", c->n_experts, DK_MAX_EXPERTS);
    if (c->n_experts > 0) {
        if (c->top_k <= 0 || c->top_k > c->n_experts || c->top_k > 16)
            return fail(DK_E_INVALID_ARG, "top_k %d with %d experts", c->top_k, c->n_experts);
        if (c->expert_ffn <= 0 || c->expert_ffn % 8)
            return fail(DK_E_UNSUPPORTED_SHAPE, "expert_ffn %d not a positive multiple of 8",
                        c->expert_ffn);
    } else if (c->ffn <= 0 || c->ffn % 8) {
        return fail(DK_E_UNSUPPORTED_SHAPE, "ffn %d not a positive multiple of 8", c->ffn);
    }
    if (!(c->rms_eps >= 0.0) || !(c->rope_theta > 0.0))
        return fail(DK_E_INVALID_ARG, "rms_eps / rope_theta out of range");
    return DK_OK;
}

}  // namespace

struct dk_kv_pool {
    dk_model_config cfg;
    int32_t num_blocks, block_size;
    uint16_t *mem;
    std::vector<int32_t> refcount;
    std::set<int32_t> free_ids;
};

struct dk_model {
    dk_model_config cfg;
    const void *embed, *lm_head, *g_final;
    std::vector<dk_layer_weights> layers;
    bool q4 = false;   // projection matrices and lm_head are packed 4-bit (dk_create_model_q4)
    double inv_freq[64];
    Profiler prof;
    // persistent step kernel: the workspace whose buffer sets hold the "not
    // written yet" pattern, which of the two sets the next step uses, step serial
    const void *fused_ws = nullptr;
    size_t fused_ws_bytes = 0;
    int fused_parity = 0;
    unsigned fused_serial = 0;
    int fused_spin_limit = dk::kFusedSpinLimit;
    long long *fused_stamps = nullptr;   // measurement aid (dk_debug_set_stage_stamps)
    int fused_stamp_layer = 0;
    int n_cus = 0;
};

namespace {

struct Workspace {
    size_t x, qkv, attn, act, cs, part, tickets, pmax_val, pmax_idx, pf_seq, total;
    size_t kpart;          // partial tiles of K-sliced GEMMs; their tickets follow the attention tickets
    int n_tickets;         // attention tickets + GEMM tickets (all cleared at the start of a step)
    // batched (matrix-core) path: activations as bf16 hi/lo, sum-of-squares partials
    size_t xhi, xlo, ahi, alo, fhi, flo, ssq;
    // mixture of experts: routing of every layer, per-row 1/rms, expert outputs
    size_t topk_idx, topk_w, rinv, yexp, rlogits, exp_cnt, exp_list;
    // persistent step kernel: two buffer sets + status words
    size_t fused_sets, fused_status;
    long long fused_set_floats;
    int fused_chunks;
    bool fused;
    int Bp;             // batch rows padded to a multiple of 16
    bool batched;
    int pack_x, pack_a, pack_f;   // batched path, inputs of K = hidden, q width and ffn: 2 or 3 terms share one 16-column operand (0: hi and lo apart)
    int chunk_tokens, max_chunks, lm_blocks;
    int pf_chunk_tokens, pf_max_chunks;   // the same split for the kernel that takes a prefill chunk's rows in groups
    bool defer_merge;   // small problems: the output projection merges the attention chunks
    bool attn_mfma;     // the matrix-core attention kernel (otherwise the vector-ALU one)
    bool attn_light;    // ... without the register double buffer (short chunks)
    bool attn_plan;     // chunks ordered on the device, from the rows' lengths (make_attn_plan)
};

constexpr int kMaxGemvBatch = 4;  // the most rows the vector-ALU GEMV takes (fewer where pack_terms, 4-bit weights or experts ask for the matrix cores)
constexpr int kLmRB = 8;     // rows per tile of the lm_head GEMV
constexpr int kLmTiles = 1;  // tiles per block of the lm_head GEMV

// The persistent step kernel is compiled for a few shape classes: (head_dim,
// query group, 512-element pieces of hidden / nq*d / ffn).  Returns the index of
// the smallest class that fits, or -1.
// Compute units of the current device, asked once per process (256 when no device answers: sizing
// calls on a machine without a GPU).  Every plan of the process uses the same number, so the workspace
// a sizing call reports always fits the launches that follow.
int device_cus()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            n = 256;
        }
        cus = n;
    }
    return cus;
}

// The persistent kernel runs one block per compute unit of the device (256 on an MI355X).
int fused_blocks() { return device_cus(); }
struct FusedClass { int d, g, ksh, ksq, ksf; };
// (0.6B-class shapes with two batch rows as well; the wide classes - 3B- and 8B-class shapes - one row)
constexpr FusedClass kFusedClasses[] = {{64, 2, 1, 1, 2}, {128, 2, 2, 4, 6}, {128, 3, 6, 6, 16}, {128, 4, 8, 8, 24}};
constexpr int kFusedTwoRowClasses = 2;
int fused_variant(const dk_model_config &c, int B)
{
    if (B > 2 || c.n_experts > 0 || c.n_layers > dk::kFusedMaxLayers) return -1;
    const int g = c.n_q_heads / c.n_kv_heads;
    // a block hands at most kFusedMaxBlockRows rows of a stage over
    const int widest = std::max(std::max((c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim, c.ffn), c.hidden);
    if ((widest + fused_blocks() - 1) / fused_blocks() > dk::kFusedMaxBlockRows) return -1;
    for (int i = 0; i < (int)(sizeof kFusedClasses / sizeof kFusedClasses[0]); i++) {
        const FusedClass &k = kFusedClasses[i];
        if (k.d == c.head_dim && k.g == g && c.hidden <= 512 * k.ksh &&
            c.n_q_heads * c.head_dim <= 512 * k.ksq && c.ffn <= 512 * k.ksf && (B == 1 || i < kFusedTwoRowClasses))
            return i;
    }
    return -1;
}

// Which kernel a batched GEMM takes (dk_gemm_plan.h: the candidate with the smallest estimated duration).
using dkplan::GemmPlan;
static_assert(dkplan::EPI_STORE == dk::GEPI_STORE && dkplan::EPI_RESID == dk::GEPI_RESID && dkplan::EPI_SWIGLU == dk::GEPI_SWIGLU,
              "the plan's epilogue codes are the kernels'");
GemmPlan gemm_plan(int epi, int N, int K, int Bp, bool q4, int pack) { return dkplan::gemm_plan(epi, N, K, Bp, q4, pack != 0, device_cus()); }
// Row blocks (= tickets) and partial-tile floats of that plan.
void gemm_plan_needs(int epi, int N, int K, int Bp, bool q4, int pack, size_t &tickets, size_t &part_floats)
{
    const GemmPlan p = gemm_plan(epi, N, K, Bp, q4, pack);
    if (p.w == 0 || p.slices == 1) return;
    const size_t tiles = (size_t)(N + 15) / 16;
    const int w = dkplan::shared_waves(epi, N, Bp / 16, p, device_cus());
    tickets = std::max(tickets, (tiles + w - 1) / w);
    part_floats = std::max(part_floats, dk::shared_gemm_part_floats(N, p.slices, epi == dk::GEPI_SWIGLU ? 2 : 1, Bp / 16));
}

// Terms of an activation that share one operand of the matrix-core GEMMs (dk_gemm.hip.h, kPackCols): two for 5..8 rows
// (and fewer of expert and 4-bit models), half the activations and products of hi and lo apart (6 rows, whole step:
// 0.6B shape 1114 -> 1010 us, 3B 2180 -> 1998, 8B 4434 -> 4019; 4 bit 3B 1651 -> 1375).
// Three or four rows of a dense model take three terms, all of float32's bits, instead of the vector-ALU products, which
// re-read float32 activations per two to four weight rows: 4 rows, 0.6B shape 1072 -> 985 us, 3B 2484 -> 1996, 8B 5208 ->
// 3809 (contexts of 512).  The vector kernel's work grows with the rows, this one's does not, so three rows gain less and
// two lose on all but the 8B shape (equal there).  Lines, by the gate matrix's bytes, whole steps, vector -> three terms:
//   * four rows from 4 MB on: 4 MB 1024 x 2048 1449 -> 1442, 2048 x 1024 1585 -> 1499, 512 x 4096 1822 -> 1833 (heads of 128)
//     and 1532 -> 1413 (of 64); 6 MB 1024 x 2816 1529 -> 1508.  Narrower layers below it gain as well (768 x 2048 1855 -> 1454).
//   * three rows from 32 MB to 256 MB: 32 MB 2048 x 8192 490 -> 477, 33 MB 3072 x 5632 452 -> 457, 34 MB 2560 x 6912 499 ->
//     495, 40 MB 2304 x 9216 472 -> 449, 50 MB (3B shape) 829 -> 815, 192 MB 6144 x 16384 596 -> 588.  Below: 22 MB 2048 x 5632
//     640 -> 646, 18 MB 1536 x 6144 740 -> 796, 6 MB (0.6B shape) 2 % slower, though 28 MB 3584 x 4096 469 -> 430.  Above: 344 MB
//     8192 x 22016 919 -> 987, 448 MB 8192 x 28672 1076 -> 1100.
constexpr int kPackRows2 = dk::kPackCols(2);
static_assert(kMaxGemvBatch <= dk::kPackCols(3), "three terms of the few-row batches fit one operand");
// Two terms go by the operand's own length K: a GEMM then takes the kernel that dk_gemm_plan_query names for its matrix,
// whatever the model's other sizes are.
int pack_terms(const dk_model_config &c, int B, bool q4, size_t K)
{
    if (K % 128 || B > kPackRows2) return 0;
    if (B > kMaxGemvBatch || c.n_experts > 0 || q4) return 2;
    const size_t H = (size_t)c.hidden, qd = (size_t)c.n_q_heads * c.head_dim;
    if (H % 128 || qd % 128 || c.ffn % 128) return 0;   // three terms: all operands or none
    const size_t mb = (H * c.ffn * 2) >> 20;   // of the gate matrix
    return B == 4 ? (mb >= 4 ? 3 : 0) : B == 3 && mb >= 32 && mb < 256 ? 3 : 0;
}

// q4: the model's matrices are 4-bit; every batch size then takes the matrix-core kernels
// allow_fused false: without the persistent kernel's hand-over buffers (they come last: everything else keeps its place)
Workspace carve(const dk_model_config &c, int B, int max_blocks, bool q4, bool allow_fused = true)
{
    Workspace w{};
    const int d = c.head_dim, G = c.n_q_heads / c.n_kv_heads;
    const size_t qkv_dim = (size_t)(c.n_q_heads + 2 * c.n_kv_heads) * d;
    const size_t act_dim = c.n_experts ? (size_t)c.top_k * c.expert_ffn : (size_t)c.ffn;
    // split the context so that rows * kv heads * chunks gives the chip a few
    // blocks per compute unit
    const int ctx_max = max_blocks * 16;
    // Which attention kernel, and how finely the context is split.  Measured:
    //  * the matrix-core kernel pays off once the group of query heads that share a kv head is
    //    large (the vector-ALU kernel's multiply-adds grow with it): from groups of 3 on; it runs
    //    best with about two blocks per compute unit, the vector-ALU one with about four;
    //  * with short chunks (at most 512 tokens: four iterations per wave) and groups of up to 4, a
    //    lighter matrix-core variant - no second set of tile registers, three blocks per compute
    //    unit, one round of at most 768 blocks - beats both (3B shape, ragged contexts up to 2 k:
    //    25.4 -> 22.5 us per launch; 0.6B shape, 16 rows of context 512: 15.1 -> 12.9 us); with 4 k
    //    contexts or groups of 8 it is slower and is not taken;
    //  * both matrix-core variants walk 128 tokens a round, so a chunk of an odd multiple of 64 leaves half of the waves
    //    idle in its last round.  The lighter one's chunks rounded down to 128 make more blocks than the chip holds where
    //    rows fill their tables and gain where they do not (whole steps, 8B shape: 16 of 2500 5400 -> 5658, of 1700 4879 ->
    //    5012, of 100 to 2300 4765 -> 4665; 4 bit, 12 of 500 to 2000 3131 -> 3034; 3B, 16 of 2400 2801 -> 2970), rounded up
    //    they gain nothing; the other's rounded up, nothing (8B, 16 of 4096 5575 / 5576).
    const bool batched_attn = B > kMaxGemvBatch || c.n_experts > 0 || q4;   // (three terms: the vector-ALU kernel's float32 probabilities)
    w.pack_x = pack_terms(c, B, q4, c.hidden);
    w.pack_a = pack_terms(c, B, q4, (size_t)c.n_q_heads * d);
    w.pack_f = c.n_experts > 0 ? 0 : pack_terms(c, B, q4, c.ffn);
    const int pairs = B * c.n_kv_heads;
    auto round64 = [](int v) { v = (v + 63) / 64 * 64; return v < 64 ? 64 : v; };
    auto chunk_for = [&](int want_blocks) {
        const int want_chunks = std::max(1, (want_blocks + pairs - 1) / pairs);
        return round64((ctx_max + want_chunks - 1) / want_chunks);
    };
    const int light_chunks = std::max(1, 768 / pairs);
    const int light_chunk = round64((ctx_max + light_chunks - 1) / light_chunks);
    int chunk;
    w.attn_mfma = w.attn_light = false;
    if (batched_attn && G >= 2 && G <= 4 && light_chunk <= 512) {
        w.attn_mfma = w.attn_light = true;
        chunk = light_chunk;
    } else if (batched_attn && G >= 3) {
        w.attn_mfma = true;
        chunk = chunk_for(512);
    } else {
        chunk = chunk_for(1024);
    }
    w.chunk_tokens = chunk;
    w.max_chunks = (ctx_max + chunk - 1) / chunk;
    w.defer_merge = false;
    // With few rows and a short context the chunk partials are a few tens of KB:
    // the output projection then merges them as it loads its input (at most 8
    // chunks, one round of loads), which saves the attention kernel a round of
    // device-wide synchronisation.
    if (B <= kMaxGemvBatch && c.n_experts == 0 && !q4 && w.pack_x != 3) {   // the vector-ALU path only
        int chunk8 = ((ctx_max + 7) / 8 + 63) / 64 * 64;
        if (chunk8 < chunk) chunk8 = chunk;
        const int n8 = (ctx_max + chunk8 - 1) / chunk8;
        if ((size_t)B * c.n_q_heads * n8 * (d + 2) * 4 <= (96u << 10) && chunk8 <= 512) {
            w.defer_merge = true;
            w.chunk_tokens = chunk8;
            w.max_chunks = n8;
        }
    }
    {
        const int rb = ((size_t)c.vocab * c.hidden * 2 < (64u << 20)) ? 2 : kLmRB;
        w.lm_blocks = (c.vocab + rb * kLmTiles - 1) / (rb * kLmTiles);
    }
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    w.x = take((size_t)B * c.hidden * 4);
    w.qkv = take((size_t)B * qkv_dim * 4);
    w.attn = take((size_t)B * c.n_q_heads * d * 4);
    w.act = take((size_t)B * act_dim * 4);
    w.cs = take((size_t)B * (d / 2) * 8);
    size_t part_floats = (size_t)B * c.n_kv_heads * w.max_chunks * G * (d + 2);
    {   // rows of a prefill chunk in groups of 16 / G: fewer, larger work items, so a finer split
        const int rpb = std::max(1, 16 / G);
        const int groups = (B + rpb - 1) / rpb;
        int want = std::max(1, 768 / (groups * c.n_kv_heads));   // three blocks per compute unit, one round
        int pchunk = ((ctx_max + want - 1) / want + 63) / 64 * 64;
        if (pchunk < 256) pchunk = 256;
        w.pf_chunk_tokens = pchunk;
        w.pf_max_chunks = (ctx_max + pchunk - 1) / pchunk;
        part_floats = std::max(part_floats, (size_t)groups * c.n_kv_heads * w.pf_max_chunks * 16 * (d + 2));
    }
    w.part = take(part_floats * 4);
    w.Bp = (B + 15) / 16 * 16;
    // expert layers and 4-bit weights use the matrix-core kernels
    w.batched = B > kMaxGemvBatch || c.n_experts > 0 || q4 || w.pack_x == 3;
    size_t gemm_tickets = 0, gemm_part = 0;
    if (w.batched) {
        const int H = c.hidden, qd = c.n_q_heads * d;
        gemm_plan_needs(dk::GEPI_STORE, (int)qkv_dim, H, w.Bp, q4, w.pack_x, gemm_tickets, gemm_part);
        gemm_plan_needs(dk::GEPI_RESID, H, qd, w.Bp, q4, w.pack_a, gemm_tickets, gemm_part);
        if (c.n_experts == 0) {
            gemm_plan_needs(dk::GEPI_SWIGLU, c.ffn, H, w.Bp, q4, w.pack_x, gemm_tickets, gemm_part);
            gemm_plan_needs(dk::GEPI_RESID, H, c.ffn, w.Bp, q4, w.pack_f, gemm_tickets, gemm_part);
        }
        gemm_plan_needs(dk::GEPI_STORE, c.vocab, H, w.Bp, q4, w.pack_x, gemm_tickets, gemm_part);
    }
    w.n_tickets = B * c.n_kv_heads + (int)gemm_tickets;
    w.tickets = take((size_t)w.n_tickets * 4);
    w.kpart = take(gemm_part * 4);
    w.pf_seq = take((size_t)DK_MAX_BATCH * 4);   // positions of a prefill chunk's rows
    if (w.batched) {
        w.lm_blocks = (c.vocab + 15) / 16;
        auto padded = [](size_t k) { return (k + 127) / 128 * 128; };   // whole K-steps
        w.xhi = take((size_t)w.Bp * padded(c.hidden) * 2);
        w.xlo = take((size_t)w.Bp * padded(c.hidden) * 2);
        w.ahi = take((size_t)w.Bp * padded((size_t)c.n_q_heads * d) * 2);
        w.alo = take((size_t)w.Bp * padded((size_t)c.n_q_heads * d) * 2);
        if (c.n_experts > 0) {
            const size_t pairs = ((size_t)B * c.top_k + 15) / 16 * 16;   // one activation row per (row, slot)
            w.fhi = take(pairs * padded((size_t)c.expert_ffn) * 2);
            w.flo = take(pairs * padded((size_t)c.expert_ffn) * 2);
            w.topk_idx = take((size_t)c.n_layers * B * c.top_k * 4);
            w.topk_w = take((size_t)B * c.top_k * 4);
            w.rinv = take((size_t)B * 4);
            w.yexp = take((size_t)B * c.top_k * c.hidden * 4);
            w.rlogits = take((size_t)B * c.n_experts * 4);
            w.exp_cnt = take((size_t)c.n_experts * 4);
            w.exp_list = take((size_t)c.n_experts * B * c.top_k * 4);
        } else {
            w.fhi = take((size_t)w.Bp * padded(act_dim) * 2);
            w.flo = take((size_t)w.Bp * padded(act_dim) * 2);
        }
        w.ssq = take((size_t)((c.hidden + 15) / 16) * dk::kSsqStride * 4);
    }
    w.pmax_val = take((size_t)B * w.lm_blocks * 4);
    w.pmax_idx = take((size_t)B * w.lm_blocks * 4);
    // (the block of a sequence's first chunk waits for the blocks of its other chunks while every block
    // works through its items in ascending order: free of cycles as long as a sequence has no more
    // chunks than there are blocks)
    w.fused = allow_fused && fused_variant(c, B) >= 0 && (ctx_max + dk::kFusedChunk - 1) / dk::kFusedChunk <= fused_blocks();
    if (w.fused) {
        w.fused_chunks = (ctx_max + dk::kFusedChunk - 1) / dk::kFusedChunk;
        w.fused_set_floats = dk::fused_layout(c.n_layers, B, c.hidden, c.n_q_heads, c.n_kv_heads, d, c.ffn,
                                              w.fused_chunks, fused_blocks()).total;
        w.fused_sets = take((size_t)2 * w.fused_set_floats * 4);
        w.fused_status = take(64);
    }
    // The plan is worth its look-up where a block's chunk takes long, and lies in the float32 attention output, which the
    // batched path does not write.
    w.attn_plan = w.batched && !w.defer_merge && w.chunk_tokens >= 256 && B * w.max_chunks <= dk::kPlanMaxItems &&
                  (B * w.max_chunks + 1) * dk::kPlanWords <= B * c.n_q_heads * d;
    w.total = off;
    return w;
}

// ---- GEMV dispatch ----------------------------------------------------------
// Rows per block tile.  Small matrices (a few MB, one or two loads per lane) are latency-bound: two rows per block
// spread them over every compute unit. Large ones (lm_head) stream better with eight rows per block.
//
// With two to four batch rows the activations are the larger stream: a thread fetches 32 bytes of x per batch row
// for every 16 bytes of a weight row, from the caches, once per weight row of its block.  From 16 MB on the rows
// per block and the threads that walk K are therefore chosen by two more rules.  Both lines come from a sweep of
// the kernel alone over weights from HBM (K = 1024..14336, 8..600 MB, 2..4 rows, about 1800 shapes, every epilogue;
// "before" is two rows and 256 threads below 64 MB, eight rows - gate/up four - and 256 threads above). Whole steps
// at 2 / 3 / 4 rows, before -> after: 3B shape (19..50 MB a matrix) 1934 / 2502 / 3011 -> 1809 / 2038 / 2520 us, 8B
// shape (33 MB and up) 3678 / 4262 / 5627 -> 3612 / 4163 / 5262; the 0.6B shape (4..6 MB) lies below the lines.
// (Those steps of 3 and 4 rows have since left this kernel, see pack_terms.  What it still has of them: sizes off the 128
// grid, three rows of layers below 32 MB and from 256 MB a gate matrix on, four rows below 4 MB.)
inline size_t gemv_bytes(const dk::GemvArgs &a) { return (size_t)a.N * a.K * 2; }
inline bool gemv_small(const dk::GemvArgs &a) { return gemv_bytes(a) < (64u << 20); }

// Four weight rows per block between 16 and 64 MB, where the blocks still fill the chip: half the activation
// traffic (before -> after, 48 MB: K = 3072, 4 rows, plain store 27.2 -> 17.1 us with the 128 threads below; K =
// 8192, 2 rows, residual 13.5 -> 12.4).  Below the line the fewer blocks cost more: K = 12288, 24 MB, 1024 weight
// rows: 18.2 -> 23.7 for gate/up; K = 2048, 17 MB: 7.3 -> 7.8. A gate/up block of two rows carries four weight rows
// already.  Another four pay at three batch rows (K = 2048, 48 MB 33.3 -> 23.3) and, at two, beyond K = 4096 (K =
// 8192, 48 MB 23.3 -> 21.7; K = 2048, 17 MB 10.2 -> 11.3). At four batch rows such a block needs 151 registers per
// lane, three waves per SIMD: it pays where the blocks are one round on the chip at least two thirds full (K =
// 4096, 6144 weight rows 34.8 -> 28.5; 7168: 39.5 -> 43.9).
inline bool gemv_four_rows(const dk::GemvArgs &a, int nb, int epi)
{
    const size_t bytes = gemv_bytes(a);
    if (nb < 2 || bytes < (16u << 20) || !gemv_small(a)) return false;
    if (a.pmax_val != nullptr) return false;   // the lm_head's grid is fixed by its table of running maxima
    if (epi == dk::EPI_SWIGLU && nb == 4) {
        if (a.K < 2048) return false;
        const int rows = a.K > 4096 ? a.N : a.N / 2;   // blocks of 256 and of 128 threads
        return rows >= 2048 && rows <= 3072;
    }
    if (a.K > 4096) return a.N >= 1600;
    if (epi == dk::EPI_SWIGLU) return nb == 3 && a.N >= 2560;
    return a.K >= 2048 && a.N >= 4096 && bytes >= (24u << 20);
}

// 128 threads instead of 256 for 2048 <= K <= 4096: a thread takes two to four strides of K instead of one or two
// (one and a half at K = 3072), so a block's fixed part - sums across lanes and waves - is shared by more of them.
// Up to 64 MB at any number of rows (0.72..1.05 of the time before).  Above 64 MB blocks of eight rows have fewer
// waves in flight with 128 threads: that loses at two batch rows (K = 2048, 200 MB, residual 35.9 -> 39.9 us) and
// at K = 4096 (3 rows, 200 MB 42.7 -> 46.7), and wins where the arithmetic weighs more: three rows below K = 4096
// (K = 2560, 200 MB 52.5 -> 45.1), four rows (K = 3584, 400 MB 139.8 -> 115.7), at K = 4096 from 10240 weight rows
// on (600 MB 189.8 -> 170.1; 64 MB 19.1 -> 21.9).
inline bool gemv_128_threads(const dk::GemvArgs &a, int nb)
{
    if (nb < 2 || a.K < 2048 || a.K > 4096 || gemv_bytes(a) < (16u << 20)) return false;
    return gemv_small(a) || (nb >= 3 && a.K < 4096) || (nb == 4 && a.N >= 10240);
}
template <int EPI>
inline int gemv_rows_per_tile(const dk::GemvArgs &a)
{
    return gemv_small(a) ? 2 : (EPI == dk::EPI_SWIGLU ? 4 : 8);
}

template <int NB, int RB, int EPI, bool NORM, bool XATTN>
dk_status launch_gemv_rb(const dk::GemvArgs &a, hipStream_t st)
{
    const int grid = (a.N + RB * a.tiles - 1) / (RB * a.tiles);
    if (a.K >= 2048 && !gemv_128_threads(a, NB))
        DK_LAUNCH(DK_K_GEMV, (dk::gemv_kernel<NB, 256, RB, EPI, NORM, XATTN>), dim3(grid), dim3(256), 0, st, a);
    else if (a.K >= 1024)
        DK_LAUNCH(DK_K_GEMV, (dk::gemv_kernel<NB, 128, RB, EPI, NORM, XATTN>), dim3(grid), dim3(128), 0, st, a);
    else
        DK_LAUNCH(DK_K_GEMV, (dk::gemv_kernel<NB, 64, RB, EPI, NORM, XATTN>), dim3(grid), dim3(64), 0, st, a);
    DK_HIP(hipGetLastError());
    return DK_OK;
}

template <int NB, int EPI, bool NORM, bool XATTN = false>
dk_status launch_gemv_nb(const dk::GemvArgs &a, hipStream_t st)
{
    if constexpr (NB >= 2)
        if (gemv_four_rows(a, NB, EPI)) return launch_gemv_rb<NB, 4, EPI, NORM, XATTN>(a, st);
    if (gemv_small(a)) return launch_gemv_rb<NB, 2, EPI, NORM, XATTN>(a, st);
    return launch_gemv_rb<NB, (EPI == dk::EPI_SWIGLU ? 4 : 8), EPI, NORM, XATTN>(a, st);
}

// y[B][N] from x[B][K]; batches above 4 rows are processed four rows at a time.
template <int EPI, bool NORM, bool XATTN = false>
dk_status launch_gemv(dk::GemvArgs a, int B, hipStream_t st)
{
    static_assert(!XATTN || (EPI == dk::EPI_RESID && !NORM), "partials feed the output projection only");
    if (a.tiles < 1) a.tiles = 1;
    const int rows_per_block = gemv_rows_per_tile<EPI>(a) * a.tiles;
    const int grid = (a.N + rows_per_block - 1) / rows_per_block;
    for (int b0 = 0; b0 < B; b0 += 4) {
        const int nb = std::min(4, B - b0);
        dk::GemvArgs g = a;
        g.x = a.x + (size_t)b0 * a.K;
        if (XATTN) {
            g.part = a.part + (size_t)b0 * a.nkv * a.max_chunks * a.group * (a.d + 2);
            g.seq_lens = a.seq_lens + b0;
        }
        g.y = a.y ? a.y + (size_t)b0 * a.N : nullptr;
        if (a.resid) g.resid = a.resid + (size_t)b0 * a.N;
        if (a.pmax_val) {
            g.pmax_val = a.pmax_val + (size_t)b0 * grid;
            g.pmax_idx = a.pmax_idx + (size_t)b0 * grid;
        }
        dk_status s;
        switch (nb) {
            case 1: s = launch_gemv_nb<1, EPI, NORM, XATTN>(g, st); break;
            case 2: s = launch_gemv_nb<2, EPI, NORM, XATTN>(g, st); break;
            case 3: s = launch_gemv_nb<3, EPI, NORM, XATTN>(g, st); break;
            default: s = launch_gemv_nb<4, EPI, NORM, XATTN>(g, st); break;
        }
        if (s != DK_OK) return s;
    }
    return DK_OK;
}

// ---- skinny GEMM dispatch (up to 64 rows; which take it: carve, pack_terms) ---
// col_groups > 1: the batch rows are split into that many groups of 16*MT across blockIdx.y
template <int MT, int KS, int RT, int EPI, bool NORM, bool KALIGNED, bool Q4 = false, int PACK = 0>
dk_status launch_gemm_inst(const dk::GemmArgs &a, int col_groups, hipStream_t st)
{
    constexpr size_t lds = dk::skinny_gemm_lds_bytes<MT, KS, RT, EPI>();
    static_assert(lds <= (64u << 10), "dynamic LDS above 64 KB would need a function attribute");
    const dim3 grid((a.N + 16 * RT - 1) / (16 * RT), col_groups);
    // K-steps in flight per wave: two (deeper did not measure faster); one where a wave has a single
    // step anyway (K <= 128 * KS: the second stage would only fetch a step it never uses - q/k/v of
    // the 0.6B shape at 16 rows 6.3 -> 5.4 us, gate/up 8.1 -> 6.8 us)
    if ((a.K + 127) / 128 <= KS) {
        DK_LAUNCH(DK_K_GEMM, (dk::skinny_gemm_kernel<MT, KS, RT, 1, EPI, NORM, KALIGNED, Q4, PACK>), grid,
                  dim3(KS * 64), lds, st, a);
    } else {
        DK_LAUNCH(DK_K_GEMM, (dk::skinny_gemm_kernel<MT, KS, RT, 2, EPI, NORM, KALIGNED, Q4, PACK>), grid,
                  dim3(KS * 64), lds, st, a);
    }
    DK_HIP(hipGetLastError());
    return DK_OK;
}

template <int MT, int KS, int RT, int EPI, bool NORM>
dk_status launch_gemm_cfg(const dk::GemmArgs &a, hipStream_t st, int col_groups = 1)
{
    if (a.pack && (MT != 1 || KS != 4 || col_groups != 1 || a.K % 128)) return fail(DK_E_INVALID_ARG, "packed terms with %d rows, K = %d", a.B, a.K);
    if (a.q4) {
        if (a.K % 128) return fail(DK_E_UNSUPPORTED_SHAPE, "4-bit matrix with K = %d (a multiple of 128 is needed)", a.K);
        if constexpr (MT == 1 && KS == 4)
            if (a.pack == 2) return launch_gemm_inst<MT, KS, RT, EPI, NORM, true, true, 2>(a, col_groups, st);
        return launch_gemm_inst<MT, KS, RT, EPI, NORM, true, true>(a, col_groups, st);
    }
    if constexpr (MT == 1 && KS == 4) {
        if (a.pack == 2) return launch_gemm_inst<MT, KS, RT, EPI, NORM, true, false, 2>(a, col_groups, st);
        if (a.pack == 3) return launch_gemm_inst<MT, KS, RT, EPI, NORM, true, false, 3>(a, col_groups, st);
    }
    if (a.K % 128 == 0) return launch_gemm_inst<MT, KS, RT, EPI, NORM, true>(a, col_groups, st);
    return launch_gemm_inst<MT, KS, RT, EPI, NORM, false>(a, col_groups, st);
}

// ---- shared-activation GEMM dispatch (see gemm_plan) -------------------------
template <int MT, int W, int EPI, bool NORM, bool Q4 = false, int PACK = 0>
dk_status launch_shared_gemm_inst(const dk::GemmArgs &a, int slices, hipStream_t st)
{
    // packed terms: what gemm_plan_16 can ask for
    if constexpr (MT == 1 && PACK == 0 && (Q4 ? EPI == dk::GEPI_STORE : EPI != dk::GEPI_STORE)) {
        if (a.pack == 2) return launch_shared_gemm_inst<MT, W, EPI, NORM, Q4, 2>(a, slices, st);
        if constexpr (!Q4)
            if (a.pack == 3) return launch_shared_gemm_inst<MT, W, EPI, NORM, Q4, 3>(a, slices, st);
    }
    if (a.pack != PACK) return fail(DK_E_INVALID_ARG, "no shared-activation GEMM for %d packed terms", a.pack);
    constexpr size_t lds = dk::shared_gemm_lds_bytes(MT);
    auto kernel = dk::shared_gemm_kernel<MT, W, 1, 2, EPI, NORM, Q4, PACK>;
    static bool lds_allowed = false;   // above 64 KB together with the kernel's static LDS: ask once
    if (!lds_allowed) {
        DK_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
        lds_allowed = true;
    }
    const int tiles = (a.N + 15) / 16;
    DK_LAUNCH(DK_K_GEMM, kernel, dim3((tiles + W - 1) / W, slices), dim3(W * 64), lds, st, a);
    DK_HIP(hipGetLastError());
    return DK_OK;
}

template <int EPI, bool NORM>
dk_status launch_shared_gemm(const dk::GemmArgs &a, int Bp, const GemmPlan &p, hipStream_t st)
{
    if (p.slices > 1 && (a.kpart == nullptr || a.ktickets == nullptr))
        return fail(DK_E_INVALID_ARG, "K-sliced GEMM without its partial buffer");
    if (p.slices < 1 || p.slices > a.K / 128) return fail(DK_E_INVALID_ARG, "%d K slices of %d columns", p.slices, a.K);
    const int mt = Bp / 16;
    if constexpr (EPI == dk::GEPI_SWIGLU) {
        if (dkplan::shared_waves(EPI, a.N, mt, p, device_cus()) == 6) {
            if (mt == 2) return a.q4 ? launch_shared_gemm_inst<2, 6, EPI, NORM, true>(a, p.slices, st) : launch_shared_gemm_inst<2, 6, EPI, NORM>(a, p.slices, st);
            if (mt == 3) return a.q4 ? launch_shared_gemm_inst<3, 6, EPI, NORM, true>(a, p.slices, st) : launch_shared_gemm_inst<3, 6, EPI, NORM>(a, p.slices, st);
            if (mt == 4) return a.q4 ? launch_shared_gemm_inst<4, 6, EPI, NORM, true>(a, p.slices, st) : launch_shared_gemm_inst<4, 6, EPI, NORM>(a, p.slices, st);
        }
    }
    if (a.q4) {
        if constexpr (EPI == dk::GEPI_RESID) {
            if (p.w == 4 && mt == 1) return launch_shared_gemm_inst<1, 4, EPI, NORM, true>(a, p.slices, st);
            if (p.w == 4 && mt == 2) return launch_shared_gemm_inst<2, 4, EPI, NORM, true>(a, p.slices, st);
            if (p.w == 4 && mt == 3) return launch_shared_gemm_inst<3, 4, EPI, NORM, true>(a, p.slices, st);
            if (p.w == 4 && mt == 4) return launch_shared_gemm_inst<4, 4, EPI, NORM, true>(a, p.slices, st);
        } else {
            if (p.w == 8 && mt == 1) return launch_shared_gemm_inst<1, 8, EPI, NORM, true>(a, p.slices, st);
            if (p.w == 8 && mt == 2) return launch_shared_gemm_inst<2, 8, EPI, NORM, true>(a, p.slices, st);
            if (p.w == 8 && mt == 3) return launch_shared_gemm_inst<3, 8, EPI, NORM, true>(a, p.slices, st);
            if (p.w == 8 && mt == 4) return launch_shared_gemm_inst<4, 8, EPI, NORM, true>(a, p.slices, st);
        }
        return fail(DK_E_INVALID_ARG, "no shared-activation 4-bit GEMM for %d rows and %d waves", Bp, p.w);
    }
    // instances: 8 waves for q | k | v, the lm_head and the gate/up pair, 4 waves for the residual
    // projections (and the gate/up pair of a large model up to 16 rows)
    if constexpr (EPI == dk::GEPI_STORE)
        if (p.w == 8 && mt == 1) return launch_shared_gemm_inst<1, 8, EPI, NORM>(a, p.slices, st);
    if constexpr (EPI == dk::GEPI_STORE || EPI == dk::GEPI_SWIGLU) {
        if (p.w == 8 && mt == 2) return launch_shared_gemm_inst<2, 8, EPI, NORM>(a, p.slices, st);
        if (p.w == 8 && mt == 3) return launch_shared_gemm_inst<3, 8, EPI, NORM>(a, p.slices, st);
        if (p.w == 8 && mt == 4) return launch_shared_gemm_inst<4, 8, EPI, NORM>(a, p.slices, st);
    }
    if constexpr (EPI == dk::GEPI_SWIGLU) {
        if (p.w == 4 && mt == 1) return launch_shared_gemm_inst<1, 4, EPI, NORM>(a, p.slices, st);
    }
    if constexpr (EPI == dk::GEPI_RESID) {
        if (p.w == 4 && mt == 1) return launch_shared_gemm_inst<1, 4, EPI, NORM>(a, p.slices, st);
        if (p.w == 4 && mt == 2) return launch_shared_gemm_inst<2, 4, EPI, NORM>(a, p.slices, st);
        if (p.w == 4 && mt == 3) return launch_shared_gemm_inst<3, 4, EPI, NORM>(a, p.slices, st);
        if (p.w == 4 && mt == 4) return launch_shared_gemm_inst<4, 4, EPI, NORM>(a, p.slices, st);
    }
    return fail(DK_E_INVALID_ARG, "no shared-activation GEMM for %d rows and %d waves", Bp, p.w);
}

template <int EPI, bool NORM>
dk_status launch_gemm(const dk::GemmArgs &a, int Bp, hipStream_t st)
{
    constexpr int NM = (EPI == dk::GEPI_SWIGLU) ? 2 : 1;
    // hidden and ffn sizes (check_config): the epilogue moves their elements in fours without a narrow path
    if (EPI != dk::GEPI_STORE && a.N % 8) return fail(DK_E_UNSUPPORTED_SHAPE, "GEMM with %d output rows (a multiple of 8 is needed)", a.N);
    const GemmPlan plan = gemm_plan(EPI, a.N, a.K, Bp, a.q4 != 0, a.pack);
    if (plan.w) return launch_shared_gemm<EPI, NORM>(a, Bp, plan, st);
    // the variant of the K-split-per-wave kernel (dk_gemm_plan.h)
    const dkplan::SkinnyVariant v = dkplan::skinny_variant(EPI, a.N, a.K, Bp, a.q4 != 0, a.pack != 0, device_cus());
#define DK_SKINNY_CASE(MT_, KS_, RT_)                                                     \
    if (v.mt == MT_ && v.ks == KS_ && v.rt == RT_) return launch_gemm_cfg<MT_, KS_, RT_, EPI, NORM>(a, st, v.groups)
    if constexpr (NM == 1) DK_SKINNY_CASE(2, 8, 2);
    if constexpr (EPI == dk::GEPI_RESID) DK_SKINNY_CASE(1, 2, 1);
    DK_SKINNY_CASE(1, 8, 1);
    DK_SKINNY_CASE(1, 8, 2);
    DK_SKINNY_CASE(1, 4, 1);
    DK_SKINNY_CASE(1, 4, 2);
    DK_SKINNY_CASE(2, 8, 1);
    DK_SKINNY_CASE(3, 4, 1);
    DK_SKINNY_CASE(4, 4, 1);
#undef DK_SKINNY_CASE
    return fail(DK_E_INVALID_ARG, "no GEMM kernel for %d rows (at most %d)", Bp, DK_MAX_BATCH);
}

// light: without the register double buffer (short chunks).  carve() takes the matrix cores for query groups of 2 to 4
// where the chunks are that short and for groups of 3 and more otherwise.
template <int D, int G, bool PLAN>
void launch_attention_mfma(const dk::AttnArgs &a, dim3 grid, bool light, hipStream_t st)
{
    if constexpr (G >= 2 && G <= 4) {
        if (light) {
            DK_LAUNCH(DK_K_ATTENTION, (dk::attention_mfma_kernel<D, G, false, PLAN>), grid, dim3(256), 0, st, a);
            return;
        }
    }
    if constexpr (G >= 3) DK_LAUNCH(DK_K_ATTENTION, (dk::attention_mfma_kernel<D, G, true, PLAN>), grid, dim3(256), 0, st, a);
}

// mfma: the matrix-core inner loop (batched path); otherwise the vector-ALU one
template <int D, bool PLAN>
dk_status launch_attention_d(const dk::AttnArgs &a, int G, dim3 grid, bool mfma, bool light, hipStream_t st)
{
#define DK_ATTN_CASE(g)                                                                              \
    case g:                                                                                          \
        if (mfma) launch_attention_mfma<D, g, PLAN>(a, grid, light, st);                             \
        else DK_LAUNCH(DK_K_ATTENTION, (dk::attention_kernel<D, g, PLAN>), grid, dim3(256), 0, st, a); \
        break;
    switch (G) {
        DK_ATTN_CASE(1)
        DK_ATTN_CASE(2)
        DK_ATTN_CASE(3)
        DK_ATTN_CASE(4)
        DK_ATTN_CASE(5)
        DK_ATTN_CASE(6)
        DK_ATTN_CASE(7)
        DK_ATTN_CASE(8)
        default: return fail(DK_E_UNSUPPORTED_SHAPE, "query group size %d", G);
    }
#undef DK_ATTN_CASE
    DK_HIP(hipGetLastError());
    return DK_OK;
}

template <int D>
dk_status launch_prefill_attention_d(const dk::AttnArgs &a, int G, dim3 grid, hipStream_t st)
{
#define DK_PF_ATTN_CASE(g)                                                                              \
    case g:                                                                                             \
        DK_LAUNCH(DK_K_ATTENTION, (dk::prefill_attention_kernel<D, g>), grid, dim3(256), 0, st, a);     \
        break;
    switch (G) {
        DK_PF_ATTN_CASE(1)
        DK_PF_ATTN_CASE(2)
        DK_PF_ATTN_CASE(3)
        DK_PF_ATTN_CASE(4)
        DK_PF_ATTN_CASE(5)
        DK_PF_ATTN_CASE(6)
        DK_PF_ATTN_CASE(7)
        DK_PF_ATTN_CASE(8)
        default: return fail(DK_E_UNSUPPORTED_SHAPE, "query group size %d", G);
    }
#undef DK_PF_ATTN_CASE
    DK_HIP(hipGetLastError());
    return DK_OK;
}

template <int NB, int D, int G, int KSH, int KSQ, int KSF, bool Q4, bool STAMPS = false>
dk_status launch_fused_q(const dk::FusedArgs &a, hipStream_t st)
{
    constexpr size_t lds = dk::fused_xs_bytes(NB, KSH, KSQ, KSF);
    auto kernel = dk::fused_step_kernel<NB, D, G, KSH, KSQ, KSF, Q4, STAMPS>;
    static bool lds_allowed = false;   // with the kernel's static LDS this can exceed 64 KB: ask once
    if (!lds_allowed) {
        DK_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
        lds_allowed = true;
    }
    DK_LAUNCH(DK_K_FUSED_STEP, kernel, dim3(fused_blocks()), dim3(dk::kFusedThreads), lds, st, a);
    DK_HIP(hipGetLastError());
    return DK_OK;
}

template <int NB, int D, int G, int KSH, int KSQ, int KSF>
dk_status launch_fused_inst(const dk::FusedArgs &a, bool q4, hipStream_t st)
{
    if (q4) return launch_fused_q<NB, D, G, KSH, KSQ, KSF, true>(a, st);
    return launch_fused_q<NB, D, G, KSH, KSQ, KSF, false>(a, st);
}

// The whole step as one persistent kernel (see dk_fused.hip.h).  Returns
// DK_E_UNSUPPORTED_SHAPE (without setting an error text) when the device cannot
// keep one block per compute unit resident; the caller then takes the ordinary path.
dk_status launch_fused(dk_model *model, dk_kv_pool *pool, const Workspace &w, char *ws,
                       const int32_t *d_block_tables, int32_t max_blocks, int32_t *d_seq_lens,
                       int32_t *d_tokens, int32_t B, float *d_logits, int32_t *d_next, bool advance,
                       hipStream_t st)
{
    const dk_model_config &c = model->cfg;
    if (model->n_cus == 0) {
        int dev = 0, n = 0;
        DK_HIP(hipGetDevice(&dev));
        DK_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        model->n_cus = n;
    }
    if (model->n_cus < fused_blocks()) return DK_E_UNSUPPORTED_SHAPE;   // (another device than the one asked first) blocks could not all be resident
    float *sets = reinterpret_cast<float *>(ws + w.fused_sets);
    unsigned *status = reinterpret_cast<unsigned *>(ws + w.fused_status);
    if (model->fused_ws != ws || model->fused_ws_bytes != w.total) {
        // first use of this workspace (or another batch shape): both sets to "not written yet"
        hipLaunchKernelGGL(dk::fused_fill_kernel, dim3(1024), dim3(256), 0, st,
                           reinterpret_cast<uint32_t *>(sets), 2 * w.fused_set_floats, status);
        DK_HIP(hipGetLastError());
        model->fused_ws = ws;
        model->fused_ws_bytes = w.total;
        model->fused_parity = 0;
    }
    dk::FusedArgs a{};
    a.L = c.n_layers;
    a.H = c.hidden;
    a.nq = c.n_q_heads;
    a.nkv = c.n_kv_heads;
    a.F = c.ffn;
    a.V = c.vocab;
    a.B = B;
    a.eps = (float)c.rms_eps;
    a.scale = (float)(1.0 / std::sqrt((double)c.head_dim));
    a.embed = static_cast<const uint16_t *>(model->embed);
    a.lm_head = static_cast<const uint16_t *>(model->lm_head);
    a.g_final = static_cast<const uint16_t *>(model->g_final);
    a.tokens = d_tokens;
    a.seq_lens = d_seq_lens;
    a.block_tables = d_block_tables;
    a.max_blocks = max_blocks;
    a.num_blocks = pool->num_blocks;
    a.pool = pool->mem;
    a.logits = d_logits;
    a.next = d_next;
    a.advance = advance ? 1 : 0;
    a.set = sets + (size_t)model->fused_parity * w.fused_set_floats;
    a.other_set = sets + (size_t)(model->fused_parity ^ 1) * w.fused_set_floats;
    a.set_floats = w.fused_set_floats;
    a.nchunks = w.fused_chunks;
    a.status = status;
    model->fused_serial = model->fused_serial + 1 == 0 ? 1 : model->fused_serial + 1;
    a.serial = model->fused_serial;
    a.spin_limit = model->fused_spin_limit;
    a.stamps = model->fused_stamps;
    a.stamp_layer = model->fused_stamp_layer;
    std::memcpy(a.inv_freq, model->inv_freq, sizeof a.inv_freq);
    for (int l = 0; l < c.n_layers; l++) {
        const dk_layer_weights &L = model->layers[(size_t)l];
        auto u16 = [](const void *p) { return static_cast<const uint16_t *>(p); };
        a.layers[l] = dk::FusedLayer{u16(L.g_attn), u16(L.w_qkv), c.qk_norm ? u16(L.g_q) : nullptr,
                                     c.qk_norm ? u16(L.g_k) : nullptr, u16(L.w_o), u16(L.g_mlp),
                                     u16(L.w_gate), u16(L.w_up), u16(L.w_down)};
    }
    model->fused_parity ^= 1;
    const int v = fused_variant(c, B);
    dk_status s = DK_E_UNSUPPORTED_SHAPE;
    if (v == 0 && B == 1) s = launch_fused_inst<1, 64, 2, 1, 1, 2>(a, model->q4, st);
    else if (v == 0 && B == 2) s = launch_fused_inst<2, 64, 2, 1, 1, 2>(a, model->q4, st);
    else if (v == 1 && B == 1 && a.stamps != nullptr && !model->q4)
        s = launch_fused_q<1, 128, 2, 2, 4, 6, false, true>(a, st);   // the one instance with stage stamps
    else if (v == 1 && B == 1) s = launch_fused_inst<1, 128, 2, 2, 4, 6>(a, model->q4, st);
    else if (v == 1 && B == 2) s = launch_fused_inst<2, 128, 2, 2, 4, 6>(a, model->q4, st);
    else if (v == 2 && B == 1) s = launch_fused_inst<1, 128, 3, 6, 6, 16>(a, model->q4, st);
    else if (v == 3 && B == 1) s = launch_fused_inst<1, 128, 4, 8, 8, 24>(a, model->q4, st);
    return s;
}

// Read-only streaming kernel of dk_read_stream: grid-stride, eight 16-byte loads in flight per lane.
__global__ __launch_bounds__(256) void read_stream_kernel(const uint4 *p, size_t n16, uint32_t *sink)
{
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    uint32_t acc = 0;
    size_t i = tid;
    for (; i + 7 * stride < n16; i += 8 * stride) {
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = p[i + u * stride];
#pragma unroll
        for (int u = 0; u < 8; u++) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (; i < n16; i += stride) {
        const uint4 v = p[i];
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    // every lane's loads feed a store that (practically) never happens: nothing can be optimised away
    if (acc == 0x9E3779B9u) sink[blockIdx.x] = acc;
}

}  // namespace

extern "C" {

const char *dk_last_error(void) { return g_err; }

// The kernel revisions change whenever a kernel's memory behaviour changes; the
// benchmark quotes stored counter measurements only for a matching revision.
const char *dk_version(void) { return "decodekit 0.9 (gfx950; gemv r4, gemm r16, attention r11, moe r4, fused r9, prefill r2, sample r4)"; }

// ------------------------------------------------------------------- pool --
dk_status dk_kv_pool_bytes(const dk_model_config *cfg, int32_t num_blocks, int32_t block_size,
                           size_t *out_bytes)
{
    dk_status s = check_config(cfg);
    if (s != DK_OK) return s;
    if (!out_bytes) return fail(DK_E_INVALID_ARG, "out_bytes is NULL");
    if (num_blocks <= 0) return fail(DK_E_INVALID_ARG, "num_blocks %d", num_blocks);
    if (block_size != 16) return fail(DK_E_UNSUPPORTED_SHAPE, "block_size %d (16 supported)", block_size);
    *out_bytes = (size_t)cfg->n_layers * num_blocks * 2 * cfg->n_kv_heads * block_size *
                 cfg->head_dim * 2;
    return DK_OK;
}

dk_status dk_create_kv_pool(const dk_model_config *cfg, int32_t num_blocks, int32_t block_size,
                            void *dev_mem, size_t dev_bytes, dk_kv_pool **out)
{
    size_t need = 0;
    dk_status s = dk_kv_pool_bytes(cfg, num_blocks, block_size, &need);
    if (s != DK_OK) return s;
    if (!out) return fail(DK_E_INVALID_ARG, "out is NULL");
    if (!dev_mem) return fail(DK_E_INVALID_ARG, "dev_mem is NULL");
    if (dev_bytes < need)
        return fail(DK_E_INVALID_ARG, "pool memory too small: %zu bytes given, %zu needed", dev_bytes, need);
    if ((uintptr_t)dev_mem % 16) return fail(DK_E_INVALID_ARG, "pool memory must be 16-byte aligned");
    dk_kv_pool *p = new (std::nothrow) dk_kv_pool;
    if (!p) return fail(DK_E_INVALID_ARG, "out of host memory");
    p->cfg = *cfg;
    p->num_blocks = num_blocks;
    p->block_size = block_size;
    p->mem = static_cast<uint16_t *>(dev_mem);
    p->refcount.assign((size_t)num_blocks, 0);
    for (int32_t i = 0; i < num_blocks; i++) p->free_ids.insert(i);
    *out = p;
    return DK_OK;
}

dk_status dk_destroy_kv_pool(dk_kv_pool *pool)
{
    delete pool;
    return DK_OK;
}

dk_status dk_kv_alloc_block(dk_kv_pool *pool, int32_t *out_block_id)
{
    if (!pool || !out_block_id) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (pool->free_ids.empty())
        return fail(DK_E_POOL_EXHAUSTED, "all %d blocks are in use", pool->num_blocks);
    const int32_t id = *pool->free_ids.begin();
    pool->free_ids.erase(pool->free_ids.begin());
    pool->refcount[(size_t)id] = 1;
    *out_block_id = id;
    return DK_OK;
}

dk_status dk_kv_alloc_block_id(dk_kv_pool *pool, int32_t block_id)
{
    if (!pool) return fail(DK_E_INVALID_ARG, "pool is NULL");
    if (block_id < 0 || block_id >= pool->num_blocks)
        return fail(DK_E_BAD_BLOCK, "block %d out of range [0,%d)", block_id, pool->num_blocks);
    if (pool->refcount[(size_t)block_id] != 0)
        return fail(DK_E_BAD_BLOCK, "block %d is in use", block_id);
    pool->free_ids.erase(block_id);
    pool->refcount[(size_t)block_id] = 1;
    return DK_OK;
}

dk_status dk_kv_retain_block(dk_kv_pool *pool, int32_t block_id)
{
    if (!pool) return fail(DK_E_INVALID_ARG, "pool is NULL");
    if (block_id < 0 || block_id >= pool->num_blocks)
        return fail(DK_E_BAD_BLOCK, "block %d out of range [0,%d)", block_id, pool->num_blocks);
    if (pool->refcount[(size_t)block_id] == 0)
        return fail(DK_E_BAD_BLOCK, "block %d is free; only a block in use can be shared", block_id);
    pool->refcount[(size_t)block_id] += 1;
    return DK_OK;
}

dk_status dk_kv_release_block(dk_kv_pool *pool, int32_t block_id)
{
    if (!pool) return fail(DK_E_INVALID_ARG, "pool is NULL");
    if (block_id < 0 || block_id >= pool->num_blocks)
        return fail(DK_E_BAD_BLOCK, "block %d out of range [0,%d)", block_id, pool->num_blocks);
    if (pool->refcount[(size_t)block_id] == 0)
        return fail(DK_E_BAD_BLOCK, "block %d is already free", block_id);
    if (--pool->refcount[(size_t)block_id] == 0) pool->free_ids.insert(block_id);
    return DK_OK;
}

dk_status dk_kv_refcount(const dk_kv_pool *pool, int32_t block_id, int32_t *out_refcount)
{
    if (!pool || !out_refcount) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (block_id < 0 || block_id >= pool->num_blocks)
        return fail(DK_E_BAD_BLOCK, "block %d out of range [0,%d)", block_id, pool->num_blocks);
    *out_refcount = pool->refcount[(size_t)block_id];
    return DK_OK;
}

dk_status dk_kv_free_blocks(const dk_kv_pool *pool, int32_t *out_free)
{
    if (!pool || !out_free) return fail(DK_E_INVALID_ARG, "NULL argument");
    *out_free = (int32_t)pool->free_ids.size();
    return DK_OK;
}

dk_status dk_kv_offset(const dk_kv_pool *pool, int32_t layer, int32_t block, int32_t kv,
                       int32_t head, int32_t slot, int32_t dim, int64_t *out_offset)
{
    if (!pool || !out_offset) return fail(DK_E_INVALID_ARG, "NULL argument");
    const dk_model_config &c = pool->cfg;
    if (layer < 0 || layer >= c.n_layers || block < 0 || block >= pool->num_blocks || kv < 0 ||
        kv > 1 || head < 0 || head >= c.n_kv_heads || slot < 0 || slot >= pool->block_size ||
        dim < 0 || dim >= c.head_dim)
        return fail(DK_E_INVALID_ARG, "pool coordinate out of range");
    *out_offset = (((((int64_t)layer * pool->num_blocks + block) * 2 + kv) * c.n_kv_heads + head) *
                       pool->block_size + slot) * c.head_dim + dim;
    return DK_OK;
}

dk_status dk_kv_validate_tables(const dk_kv_pool *pool, const int32_t *bt, int32_t max_blocks,
                                const int32_t *seq_lens, int32_t B)
{
    if (!pool || !bt || !seq_lens) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (B <= 0 || max_blocks <= 0) return fail(DK_E_INVALID_ARG, "B %d, max_blocks_per_seq %d", B, max_blocks);
    std::set<int32_t> targets;
    for (int32_t b = 0; b < B; b++) {
        const int32_t T = seq_lens[b];
        if (T < 0 || T / pool->block_size >= max_blocks)
            return fail(DK_E_INVALID_ARG, "row %d: seq_len %d does not fit %d blocks of %d", b, T,
                        max_blocks, pool->block_size);
        const int32_t last = T / pool->block_size;
        for (int32_t i = 0; i <= last; i++) {
            const int32_t id = bt[(size_t)b * max_blocks + i];
            if (id < 0 || id >= pool->num_blocks)
                return fail(DK_E_BAD_BLOCK, "row %d, table entry %d: block %d out of range [0,%d)", b,
                            i, id, pool->num_blocks);
            if (pool->refcount[(size_t)id] == 0)
                return fail(DK_E_BAD_BLOCK, "row %d, table entry %d: block %d is free", b, i, id);
        }
        const int32_t tgt = bt[(size_t)b * max_blocks + last];
        if (pool->refcount[(size_t)tgt] != 1)
            return fail(DK_E_BAD_BLOCK, "row %d: append target block %d is shared (refcount %d)", b,
                        tgt, pool->refcount[(size_t)tgt]);
        if (!targets.insert(tgt).second)
            return fail(DK_E_BAD_BLOCK, "row %d: append target block %d is also another row's", b, tgt);
    }
    return DK_OK;
}

dk_status dk_append_kv(dk_kv_pool *pool, int32_t layer, const int32_t *d_block_tables,
                       int32_t max_blocks, const int32_t *d_seq_lens, int32_t B, const void *d_k,
                       const void *d_v, void *hip_stream)
{
    if (!pool || !d_block_tables || !d_seq_lens || !d_k || !d_v)
        return fail(DK_E_INVALID_ARG, "NULL argument");
    if (layer < 0 || layer >= pool->cfg.n_layers) return fail(DK_E_INVALID_ARG, "layer %d", layer);
    if (B <= 0 || B > DK_MAX_BATCH) return fail(DK_E_INVALID_ARG, "B %d (1..%d)", B, DK_MAX_BATCH);
    if (max_blocks <= 0) return fail(DK_E_INVALID_ARG, "max_blocks_per_seq %d", max_blocks);
    dk::AppendArgs a{static_cast<const uint16_t *>(d_k), static_cast<const uint16_t *>(d_v),
                     pool->mem, d_block_tables, d_seq_lens, max_blocks, pool->num_blocks,
                     pool->block_size, layer, pool->cfg.n_kv_heads, pool->cfg.head_dim};
    hipLaunchKernelGGL(dk::append_kv_kernel, dim3(pool->cfg.n_kv_heads, B, 2), dim3(128), 0,
                       static_cast<hipStream_t>(hip_stream), a);
    DK_HIP(hipGetLastError());
    return DK_OK;
}

// ------------------------------------------------------------------ model --
dk_status dk_create_model(const dk_model_config *cfg, const dk_weight_ptrs *w, dk_model **out)
{
    dk_status s = check_config(cfg);
    if (s != DK_OK) return s;
    if (!w || !out) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (!w->embed || !w->lm_head || !w->g_final || !w->layers)
        return fail(DK_E_INVALID_ARG, "a top-level weight pointer is NULL");
    if (cfg->n_experts > 0 && cfg->hidden > 8192)
        return fail(DK_E_UNSUPPORTED_SHAPE, "mixture-of-experts layers support hidden <= 8192 (got %d)",
                    cfg->hidden);
    for (int l = 0; l < cfg->n_layers; l++) {
        const dk_layer_weights &L = w->layers[l];
        if (!L.g_attn || !L.w_qkv || !L.w_o || !L.g_mlp || !L.w_gate || !L.w_up || !L.w_down)
            return fail(DK_E_INVALID_ARG, "layer %d: a weight pointer is NULL", l);
        if (cfg->qk_norm && (!L.g_q || !L.g_k))
            return fail(DK_E_INVALID_ARG, "layer %d: qk_norm set but g_q / g_k is NULL", l);
        if (cfg->n_experts > 0 && !L.w_router)
            return fail(DK_E_INVALID_ARG, "layer %d: w_router is NULL", l);
    }
    dk_model *m = new (std::nothrow) dk_model;
    if (!m) return fail(DK_E_INVALID_ARG, "out of host memory");
    m->cfg = *cfg;
    m->embed = w->embed;
    m->lm_head = w->lm_head;
    m->g_final = w->g_final;
    m->layers.assign(w->layers, w->layers + cfg->n_layers);
    const int half = cfg->head_dim / 2;
    for (int i = 0; i < 64; i++)
        m->inv_freq[i] = i < half ? std::pow(cfg->rope_theta, -2.0 * i / cfg->head_dim) : 0.0;
    *out = m;
    return DK_OK;
}

dk_status dk_create_model_q4(const dk_model_config *cfg, const dk_weight_ptrs *w, dk_model **out)
{
    dk_status s = check_config(cfg);
    if (s != DK_OK) return s;
    const int qd = cfg->n_q_heads * cfg->head_dim;
    const int width = cfg->n_experts > 0 ? cfg->expert_ffn : cfg->ffn;
    if (cfg->hidden % 128 || qd % 128 || width % 128)
        return fail(DK_E_UNSUPPORTED_SHAPE,
                    "4-bit weights need hidden, n_q_heads*head_dim and the MLP width to be multiples of 128 "
                    "(got %d, %d, %d)", cfg->hidden, qd, width);
    if (cfg->n_experts > 0 && (cfg->hidden < 512 || cfg->expert_ffn < 512))
        return fail(DK_E_UNSUPPORTED_SHAPE, "4-bit experts need hidden and expert_ffn of at least 512 (got %d, %d)",
                    cfg->hidden, cfg->expert_ffn);
    if (w && w->embed && w->embed == w->lm_head)
        return fail(DK_E_INVALID_ARG, "the embedding stays bf16 and cannot double as the 4-bit lm_head");
    if ((s = dk_create_model(cfg, w, out)) != DK_OK) return s;
    (*out)->q4 = true;
    return DK_OK;
}

dk_status dk_destroy_model(dk_model *model)
{
    if (model) {
        // a later model at the same address must not pass for the last user of the static scratch
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        for (auto &o : g_scratch_owner)
            if (o == model) o = nullptr;
    }
    delete model;
    return DK_OK;
}

dk_status dk_workspace_bytes(const dk_model *model, int32_t max_B, int32_t max_blocks,
                             size_t *out_bytes)
{
    if (!model || !out_bytes) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (max_B <= 0 || max_B > DK_MAX_BATCH) return fail(DK_E_INVALID_ARG, "max_B %d (1..%d)", max_B, DK_MAX_BATCH);
    if (max_blocks <= 0) return fail(DK_E_INVALID_ARG, "max_blocks_per_seq %d", max_blocks);
    // the layout depends on the batch size (which kernels run, which buffers they need): a workspace
    // "for batches up to max_B" has to hold the largest of them
    size_t need = 0;
    for (int b = 1; b <= max_B; b++) need = std::max(need, carve(model->cfg, b, max_blocks, model->q4).total);
    *out_bytes = need;
    return DK_OK;
}

// internal to this file: the rows are consecutive positions of one sequence (chunked prefill)
constexpr uint32_t kStepPrefill = 0x80000000u;

static dk_status decode_step_impl(dk_model *model, dk_kv_pool *pool, const int32_t *d_block_tables,
                                  int32_t max_blocks, int32_t *d_seq_lens, int32_t *d_tokens, int32_t B,
                                  void *d_workspace, size_t workspace_bytes, float *d_logits,
                                  int32_t *d_next_tokens, uint32_t flags, void *hip_stream);

dk_status dk_decode_step(dk_model *model, dk_kv_pool *pool, const int32_t *d_block_tables,
                         int32_t max_blocks, int32_t *d_seq_lens, int32_t *d_tokens, int32_t B,
                         void *d_workspace, size_t workspace_bytes, float *d_logits,
                         int32_t *d_next_tokens, uint32_t flags, void *hip_stream)
{
    if (!model) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (!(flags & DK_STEP_PROFILE))
        return decode_step_impl(model, pool, d_block_tables, max_blocks, d_seq_lens, d_tokens, B,
                                d_workspace, workspace_bytes, d_logits, d_next_tokens, flags, hip_stream);
    // profiled step: every launch carries its own start/stop events; the stream
    // is synchronised afterwards and the times are added to the model's totals
    Profiler &p = model->prof;
    g_prof = &p;
    const dk_status s = decode_step_impl(model, pool, d_block_tables, max_blocks, d_seq_lens, d_tokens,
                                         B, d_workspace, workspace_bytes, d_logits, d_next_tokens,
                                         flags & ~DK_STEP_PROFILE, hip_stream);
    g_prof = nullptr;
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(hip_stream));
    for (auto &q : p.pending) {
        float ms = 0.f;
        if (e == hipSuccess && hipEventElapsedTime(&ms, q.e0, q.e1) == hipSuccess) {
            p.ms[q.cls] += ms;
            p.launches[q.cls] += 1;
        }
        p.free_events.push_back(q.e0);
        p.free_events.push_back(q.e1);
    }
    p.pending.clear();
    if (s != DK_OK) return s;
    if (e != hipSuccess) return fail(DK_E_HIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
    return DK_OK;
}

dk_status dk_decode_step_static(dk_model *model, dk_kv_pool *pool, const int32_t *d_block_tables,
                                int32_t max_blocks, int32_t *d_seq_lens, int32_t *d_tokens, int32_t B,
                                float *d_logits, int32_t *d_next_tokens, uint32_t flags, void *hip_stream)
{
    if (!model) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (flags & DK_STEP_PROFILE)
        return fail(DK_E_INVALID_ARG, "DK_STEP_PROFILE creates events; the entry point that allocates nothing refuses it");
    if (B <= 0 || B > DK_MAX_BATCH) return fail(DK_E_INVALID_ARG, "B %d (1..%d)", B, DK_MAX_BATCH);
    if (max_blocks <= 0) return fail(DK_E_INVALID_ARG, "max_blocks_per_seq %d", max_blocks);
    size_t need = carve(model->cfg, B, max_blocks, model->q4, !(flags & DK_STEP_NO_FUSED)).total;
    if (need > DK_STATIC_SCRATCH_BYTES && !(flags & DK_STEP_NO_FUSED)) {
        // the persistent kernel's hand-over buffers (two sets, every layer's attention partials) outgrow the
        // array for long tables of the wide shapes: such a step runs one kernel per stage instead
        flags |= DK_STEP_NO_FUSED;
        need = carve(model->cfg, B, max_blocks, model->q4, false).total;
    }
    if (need > DK_STATIC_SCRATCH_BYTES)
        return fail(DK_E_WORKSPACE_TOO_SMALL,
                    "this step needs %zu bytes of workspace; the static scratch holds %zu (use dk_decode_step "
                    "with a caller-owned workspace)", need, (size_t)DK_STATIC_SCRATCH_BYTES);
    int dev = 0;
    DK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(DK_E_INVALID_ARG, "device index %d (below %d)", dev, kMaxDevices);
    void *ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (g_scratch_ptr[dev] == nullptr) {
            // once per GPU, with that GPU current: the address of its copy of the array
            void *p = nullptr;
            DK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            if (p == nullptr || (uintptr_t)p % 256) return fail(DK_E_HIP, "static scratch has no usable device address");
            g_scratch_ptr[dev] = p;
        }
        ws = g_scratch_ptr[dev];
        if (g_scratch_owner[dev] != model) {
            // someone else's step has been through the array since this model's last one (or this
            // is its first): whatever the persistent kernel had prepared there is gone
            if (model->fused_ws == ws) model->fused_ws = nullptr;
            g_scratch_owner[dev] = model;
        }
    }
    return decode_step_impl(model, pool, d_block_tables, max_blocks, d_seq_lens, d_tokens, B, ws,
                            DK_STATIC_SCRATCH_BYTES, d_logits, d_next_tokens, flags, hip_stream);
}

dk_status dk_prefill_chunk(dk_model *model, dk_kv_pool *pool, const int32_t *d_block_table,
                           int32_t max_blocks, int32_t start, const int32_t *d_tokens, int32_t n,
                           void *d_workspace, size_t workspace_bytes, float *d_logits,
                           int32_t *d_next_tokens, void *hip_stream)
{
    if (!model || !pool || !d_block_table || !d_tokens || !d_workspace || (!d_next_tokens && d_logits))
        return fail(DK_E_INVALID_ARG, "NULL argument");
    if (n <= 0 || n > DK_MAX_BATCH) return fail(DK_E_INVALID_ARG, "chunk of %d tokens (1..%d)", n, DK_MAX_BATCH);
    if (max_blocks <= 0) return fail(DK_E_INVALID_ARG, "max_blocks %d", max_blocks);
    if (start < 0 || (int64_t)start + n > (int64_t)max_blocks * pool->block_size)
        return fail(DK_E_INVALID_ARG, "positions %d..%d do not fit a table of %d blocks", start, start + n - 1,
                    max_blocks);
    if ((uintptr_t)d_workspace % 256) return fail(DK_E_INVALID_ARG, "workspace must be 256-byte aligned");
    const Workspace w = carve(model->cfg, n, max_blocks, model->q4);
    if (workspace_bytes < w.total)
        return fail(DK_E_WORKSPACE_TOO_SMALL, "workspace %zu bytes, %zu needed", workspace_bytes, w.total);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int *seq = reinterpret_cast<int *>(static_cast<char *>(d_workspace) + w.pf_seq);
    hipLaunchKernelGGL(dk::iota_kernel, dim3(1), dim3(64), 0, st, seq, start, n);
    DK_HIP(hipGetLastError());
    // the step neither advances nor writes the tokens, so the cast is safe
    return decode_step_impl(model, pool, d_block_table, max_blocks, seq, const_cast<int32_t *>(d_tokens), n,
                            d_workspace, workspace_bytes, d_logits, d_next_tokens,
                            DK_STEP_NO_FUSED | kStepPrefill, hip_stream);
}

namespace {
struct SampleScratch { size_t p, pmax, part, hist, st_a, st_b, item_val, item_cnt, total; };
SampleScratch sample_scratch(int B, int V)
{
    SampleScratch L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off = align_up(off + bytes, 256); return o; };
    L.p = take((size_t)B * V * 4);
    L.pmax = take((size_t)B * dk::kSampleBlocks * 4);
    L.part = take((size_t)B * dk::kSampleBlocks * 4);
    L.st_a = take((size_t)B * sizeof(dk::SampleState));
    L.st_b = take((size_t)B * sizeof(dk::SampleState));
    L.item_val = take((size_t)B * dk::kSampleItems * 4);
    L.item_cnt = take((size_t)B * dk::kSampleItems * 4);
    L.total = off;
    L.hist = L.item_val;   // the searches' histograms, where the selection path has its items
    static_assert(3 * dk::kSampleBins * sizeof(unsigned long long) <= 2 * dk::kSampleItems * 4, "three histograms a row");
    return L;
}
}  // namespace

dk_status dk_sample_scratch_bytes(int32_t B, int32_t V, size_t *out_bytes)
{
    if (!out_bytes) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (B <= 0 || V <= 0) return fail(DK_E_INVALID_ARG, "B %d, V %d", B, V);
    *out_bytes = sample_scratch(B, V).total;
    return DK_OK;
}

dk_status dk_sample_tokens(const float *d_logits, int32_t B, int32_t V, const dk_sampling *params,
                           uint64_t step, void *d_scratch, size_t scratch_bytes, int32_t *d_out,
                           void *hip_stream)
{
    if (!d_logits || !params || !d_scratch || !d_out) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (B <= 0 || V <= 0) return fail(DK_E_INVALID_ARG, "B %d, V %d", B, V);
    if (!(params->temperature > 0.f)) return fail(DK_E_INVALID_ARG, "temperature must be positive");
    if (params->top_k < 0) return fail(DK_E_INVALID_ARG, "top_k %d", params->top_k);
    if (!(params->top_p > 0.f && params->top_p <= 1.f)) return fail(DK_E_INVALID_ARG, "top_p outside (0, 1]");
    if ((uintptr_t)d_scratch % 256) return fail(DK_E_INVALID_ARG, "scratch must be 256-byte aligned");
    const SampleScratch L = sample_scratch(B, V);
    if (scratch_bytes < L.total)
        return fail(DK_E_WORKSPACE_TOO_SMALL, "scratch %zu bytes, %zu needed", scratch_bytes, L.total);
    char *base = static_cast<char *>(d_scratch);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    dk::SampleArgs a{};
    a.logits = d_logits;
    a.p = reinterpret_cast<float *>(base + L.p);
    a.pmax = reinterpret_cast<float *>(base + L.pmax);
    a.out = d_out;
    a.V = V;
    a.temperature = params->temperature;
    a.top_p = params->top_p;
    a.top_k = params->top_k;
    a.seed_lo = (uint32_t)params->seed;
    a.seed_hi = (uint32_t)(params->seed >> 32);
    a.step_lo = (uint32_t)step;
    a.step_hi = (uint32_t)(step >> 32);
    a.part = reinterpret_cast<float *>(base + L.part);
    // totals of V weights of at most 1 are at most 2^63
    a.mass_bits = 63;
    for (int n = V; n > 1; n = (n + 1) / 2) a.mass_bits--;
    dk::SampleState *state[2] = {reinterpret_cast<dk::SampleState *>(base + L.st_a),
                                 reinterpret_cast<dk::SampleState *>(base + L.st_b)};
    // three histograms in turn: the one the last launch added to, the one this launch adds to, the one it clears
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(base + L.hist);
    const size_t hist_words = (size_t)B * dk::kSampleBins;
    int n_launch = 0;
    auto launch = [&](void (*kernel)(dk::SampleArgs), int grid_x) {
        a.st_in = state[n_launch & 1];
        a.st_out = state[(n_launch & 1) ^ 1];
        a.hist_in = hist + (size_t)((n_launch + 2) % 3) * hist_words;
        a.hist_out = hist + (size_t)(n_launch % 3) * hist_words;
        a.hist_clear = hist + (size_t)((n_launch + 1) % 3) * hist_words;
        hipLaunchKernelGGL(kernel, dim3(grid_x, B), dim3(dk::kSampleThreads), 0, st, a);
        n_launch++;
    };
    const bool use_k = params->top_k > 0 && params->top_k < V, use_p = params->top_p < 1.f;
    const bool select = use_k && params->top_k <= dk::kSampleFastK && V <= dk::kSampleBlocks * dk::kSampleSliceMax;
    a.search = (use_k || use_p) && !select;
    a.count = use_k;
    a.negligible = use_k ? 0.f : (1.f - params->top_p) / (2.f * (float)V);
    launch(dk::sample_max_kernel, dk::kSampleBlocks);
    if (select) {
        // few candidates: the weights and the slices' top k, then one block per row for thresholds and draw
        dk::SampleSelectArgs s{};
        s.logits = d_logits;
        s.p = a.p;
        s.pmax = a.pmax;
        s.item_val = reinterpret_cast<float *>(base + L.item_val);
        s.item_cnt = reinterpret_cast<uint32_t *>(base + L.item_cnt);
        s.out = d_out;
        s.V = V;
        s.top_k = params->top_k;
        s.temperature = params->temperature;
        s.top_p = params->top_p;
        s.seed_lo = a.seed_lo;
        s.seed_hi = a.seed_hi;
        s.step_lo = a.step_lo;
        s.step_hi = a.step_hi;
        hipLaunchKernelGGL(dk::sample_exp_topk_kernel, dim3(dk::kSampleBlocks, B), dim3(dk::kSampleThreads), 0, st, s);
        hipLaunchKernelGGL(dk::sample_merge_draw_kernel, dim3(1, B), dim3(dk::kSampleThreads), 0, st, s);
        DK_HIP(hipGetLastError());
        return DK_OK;
    }
    // a search: a launch per digit makes its histogram (the first: the launch that makes the weights, or the one that
    // settles the top-k threshold), the next one settles it
    auto later_digits = [&](bool count) {
        a.count = a.count_in = count;
        for (int shift = dk::kSampleTopShift - dk::kSampleDigitBits; shift >= 0; shift -= dk::kSampleDigitBits) {
            a.shift = shift;
            a.first = shift == dk::kSampleTopShift - dk::kSampleDigitBits;
            launch(dk::sample_kernel<dk::SAMPLE_PASS>, dk::kSampleBlocks);
        }
        a.first = 0;
    };
    launch(a.search ? dk::sample_kernel<dk::SAMPLE_EXP_DIGIT> : dk::sample_kernel<dk::SAMPLE_EXP>, dk::kSampleBlocks);
    if (!a.search) {
        launch(dk::sample_kernel<dk::SAMPLE_DRAW>, 1);
        DK_HIP(hipGetLastError());
        return DK_OK;
    }
    if (use_k) later_digits(true);
    if (use_k && use_p) {
        a.second = 1;
        a.count = 0;
        a.shift = dk::kSampleTopShift;
        launch(dk::sample_kernel<dk::SAMPLE_PASS>, dk::kSampleBlocks);
        a.second = 0;
    }
    if (use_p) later_digits(false);
    launch(dk::sample_kernel<dk::SAMPLE_KEEP>, dk::kSampleBlocks);
    launch(dk::sample_kernel<dk::SAMPLE_DRAW>, 1);
    DK_HIP(hipGetLastError());
    return DK_OK;
}

dk_status dk_profile_read(dk_model *model, double *out_ms, int64_t *out_launches, int32_t reset)
{
    if (!model || !out_ms || !out_launches) return fail(DK_E_INVALID_ARG, "NULL argument");
    for (int i = 0; i < DK_K_COUNT; i++) {
        out_ms[i] = model->prof.ms[i];
        out_launches[i] = model->prof.launches[i];
        if (reset) { model->prof.ms[i] = 0.0; model->prof.launches[i] = 0; }
    }
    return DK_OK;
}

static dk_status decode_step_impl(dk_model *model, dk_kv_pool *pool, const int32_t *d_block_tables,
                                  int32_t max_blocks, int32_t *d_seq_lens, int32_t *d_tokens, int32_t B,
                                  void *d_workspace, size_t workspace_bytes, float *d_logits,
                                  int32_t *d_next_tokens, uint32_t flags, void *hip_stream)
{
    if (!model || !pool || !d_block_tables || !d_seq_lens || !d_tokens || !d_workspace ||
        (!d_next_tokens && !(flags & kStepPrefill)))
        return fail(DK_E_INVALID_ARG, "NULL argument");
    if (B <= 0 || B > DK_MAX_BATCH) return fail(DK_E_INVALID_ARG, "B %d (1..%d)", B, DK_MAX_BATCH);
    if (max_blocks <= 0) return fail(DK_E_INVALID_ARG, "max_blocks_per_seq %d", max_blocks);
    if (flags & ~(DK_STEP_ADVANCE | DK_STEP_NO_FUSED | kStepPrefill))
        return fail(DK_E_INVALID_ARG, "unknown flags 0x%x", flags);
    const bool prefill = (flags & kStepPrefill) != 0;
    const dk_model_config &c = model->cfg;
    const dk_model_config &pc = pool->cfg;
    if (pc.n_layers != c.n_layers || pc.n_kv_heads != c.n_kv_heads || pc.head_dim != c.head_dim)
        return fail(DK_E_INVALID_ARG, "pool was created for a different model shape");
    if ((uintptr_t)d_workspace % 256) return fail(DK_E_INVALID_ARG, "workspace must be 256-byte aligned");
    const Workspace w = carve(c, B, max_blocks, model->q4, !(flags & DK_STEP_NO_FUSED));
    if (workspace_bytes < w.total)
        return fail(DK_E_WORKSPACE_TOO_SMALL, "workspace %zu bytes, %zu needed", workspace_bytes, w.total);

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(d_workspace);
    if (w.fused) {
        const dk_status fs = launch_fused(model, pool, w, ws, d_block_tables, max_blocks, d_seq_lens, d_tokens,
                                          B, d_logits, d_next_tokens, (flags & DK_STEP_ADVANCE) != 0, st);
        if (fs != DK_E_UNSUPPORTED_SHAPE) return fs;   // otherwise: the ordinary path below
    }
    // a step of another shape lays the workspace out differently and overwrites the
    // persistent kernel's hand-over buffers: its next use starts from scratch
    if (model->fused_ws == ws && model->fused_ws_bytes != w.total) model->fused_ws = nullptr;
    float *x = reinterpret_cast<float *>(ws + w.x);
    float *qkv = reinterpret_cast<float *>(ws + w.qkv);
    float *attn = reinterpret_cast<float *>(ws + w.attn);
    float *act = reinterpret_cast<float *>(ws + w.act);
    float2 *cs = reinterpret_cast<float2 *>(ws + w.cs);
    float *part = reinterpret_cast<float *>(ws + w.part);
    int *tickets = reinterpret_cast<int *>(ws + w.tickets);
    float *kpart = reinterpret_cast<float *>(ws + w.kpart);
    int *ktickets = tickets + B * c.n_kv_heads;   // behind the attention tickets, cleared with them
    float *pmax_val = reinterpret_cast<float *>(ws + w.pmax_val);
    int *pmax_idx = reinterpret_cast<int *>(ws + w.pmax_idx);
    uint16_t *xhi = reinterpret_cast<uint16_t *>(ws + w.xhi), *xlo = reinterpret_cast<uint16_t *>(ws + w.xlo);
    uint16_t *ahi = reinterpret_cast<uint16_t *>(ws + w.ahi), *alo = reinterpret_cast<uint16_t *>(ws + w.alo);
    uint16_t *fhi = reinterpret_cast<uint16_t *>(ws + w.fhi), *flo = reinterpret_cast<uint16_t *>(ws + w.flo);
    uint16_t *x3 = nullptr, *a3 = nullptr, *f3 = nullptr;
    // packed: the other terms lie in further columns of the first one's operand
    auto next = [](int terms) { return dk::kPackCols(terms) * 8; };
    if (w.pack_x) xlo = xhi + next(w.pack_x);
    if (w.pack_a) alo = ahi + next(w.pack_a);
    if (w.pack_f) flo = fhi + next(w.pack_f);
    if (w.pack_x == 3) { x3 = xlo + next(3); a3 = alo + next(3); f3 = flo + next(3); }
    float *ssq = reinterpret_cast<float *>(ws + w.ssq);

    const int H = c.hidden, d = c.head_dim, nq = c.n_q_heads, nkv = c.n_kv_heads;
    const int qkv_dim = (nq + 2 * nkv) * d;
    const float eps = (float)c.rms_eps;
    const bool batched = w.batched;
    const int ssq_tiles = (H + 15) / 16;   // sum-of-squares partials a residual GEMM leaves
    dk_status s;
    auto u16 = [](const void *p) { return static_cast<const uint16_t *>(p); };

    // The chunk's k and v reach the pool from the projection itself where its blocks hold a head each.
    const bool grouped = prefill && batched && w.pack_x != 3;   // attention takes 16 / G rows of the sequence together
    const bool qkv_appends = grouped && d == 128 && H % 128 == 0 &&
                             gemm_plan(dk::GEPI_STORE, qkv_dim, H, w.Bp, model->q4, w.pack_x).w == 8;
    // A prefill chunk whose predictions nobody wants (all but the last of a prompt) leaves K/V and, in a model with
    // experts, the routing: it ends with the last layer's (501 tokens of the 8B shape: 7 of 8 chunks, 2 % of the call).
    const bool kv_only = prefill && d_next_tokens == nullptr && d_logits == nullptr;
    uint32_t *plan = w.attn_plan && !prefill ? reinterpret_cast<uint32_t *>(attn) : nullptr;
    {   // embedding rows, rotary angles, cleared tickets
        dk::EmbedArgs e{};
        e.embed = u16(model->embed);
        e.tokens = d_tokens;
        e.seq_lens = d_seq_lens;
        e.x = x;
        e.cs = cs;
        e.tickets = tickets;
        e.n_tickets = w.n_tickets;
        e.B = B;
        if (plan) {
            e.plan = plan;
            e.plan_items = B * w.max_chunks;
            e.plan_chunk = w.chunk_tokens;
            e.plan_chunks = w.max_chunks;
            e.block_tables = d_block_tables;
            e.max_blocks = max_blocks;
        }
        e.H = H;
        e.half = d / 2;
        e.V = c.vocab;
        if (batched) {
            e.gain = u16(model->layers[0].g_attn);
            e.xhi = xhi;
            e.xlo = xlo;
            e.x3 = x3;
            e.ssq_out = ssq;
        }
        std::memcpy(e.inv_freq, model->inv_freq, sizeof e.inv_freq);
        DK_LAUNCH(DK_K_EMBED, dk::embed_kernel, dim3(plan ? B + 1 : B), dim3(256), 0, st, e);
        DK_HIP(hipGetLastError());
    }

    for (int l = 0; l < c.n_layers; l++) {
        const dk_layer_weights &L = model->layers[(size_t)l];
        // q, k, v = W_qkv * rmsnorm(x)
        if (batched) {
            dk::GemmArgs g{};
            g.W = u16(L.w_qkv);
            g.N = qkv_dim;
            g.K = H;
            g.B = B;
            g.q4 = model->q4;
            g.pack = w.pack_x;
            g.kpart = kpart;
            g.ktickets = ktickets;
            g.xhi = xhi;
            g.xlo = xlo;
            g.ssq_in = ssq;
            // who wrote the partials: the embedding (1), the expert combine, or a residual GEMM
            g.n_part = (l == 0) ? 1 : (c.n_experts > 0) ? (H + 1023) / 1024 : ssq_tiles;
            g.eps = eps;
            g.y = qkv;
            if (qkv_appends) {
                g.q_heads = nq;
                g.kv_heads = nkv;
                g.cs = cs;
                g.g_k = c.qk_norm ? u16(L.g_k) : nullptr;
                g.pool = pool->mem;
                g.block_table = d_block_tables;
                g.seq_lens = d_seq_lens;
                g.max_blocks = max_blocks;
                g.num_blocks = pool->num_blocks;
                g.layer = l;
            }
            if ((s = launch_gemm<dk::GEPI_STORE, true>(g, w.Bp, st)) != DK_OK) return s;
        } else {
            dk::GemvArgs g{};
            g.W = u16(L.w_qkv);
            g.x = x;
            g.gain = u16(L.g_attn);
            g.eps = eps;
            g.y = qkv;
            g.N = qkv_dim;
            g.K = H;
            if ((s = launch_gemv<dk::EPI_STORE, true>(g, B, st)) != DK_OK) return s;
        }
        {   // head norm, rotation, KV append and attention over positions 0..T
            dk::AttnArgs a{};
            a.qkv = qkv;
            a.cs = cs;
            a.g_q = c.qk_norm ? u16(L.g_q) : nullptr;
            a.g_k = c.qk_norm ? u16(L.g_k) : nullptr;
            a.pool = pool->mem;
            a.block_tables = d_block_tables;
            a.seq_lens = d_seq_lens;
            a.out = attn;
            if (batched) {
                a.out_hi = ahi;
                a.out_lo = alo;
                a.out_x3 = a3;
            }
            a.part = part;
            a.tickets = tickets;
            a.max_blocks = max_blocks;
            a.num_blocks = pool->num_blocks;
            a.layer = l;
            a.nq = nq;
            a.nkv = nkv;
            a.chunk_tokens = w.chunk_tokens;
            a.max_chunks = w.max_chunks;
            a.defer_merge = w.defer_merge ? 1 : 0;
            a.table_stride = prefill ? 0 : max_blocks;
            a.no_append = prefill ? 1 : 0;
            const bool append_only = l + 1 == c.n_layers && kv_only && c.n_experts == 0;
            if (prefill && !qkv_appends) {
                dk::PrefillAppendArgs pa{};
                pa.qkv = qkv;
                pa.cs = cs;
                pa.g_k = a.g_k;
                pa.pool = pool->mem;
                pa.block_table = d_block_tables;
                pa.seq_lens = d_seq_lens;
                pa.max_blocks = max_blocks;
                pa.num_blocks = pool->num_blocks;
                pa.layer = l;
                pa.nq = nq;
                pa.nkv = nkv;
                pa.eps = eps;
                if (d == 128) {
                    DK_LAUNCH(DK_K_ATTENTION, dk::prefill_append_kernel<128>, dim3(B), dim3(256), 0, st, pa);
                } else {
                    DK_LAUNCH(DK_K_ATTENTION, dk::prefill_append_kernel<64>, dim3(B), dim3(256), 0, st, pa);
                }
                DK_HIP(hipGetLastError());
            }
            if (append_only) return DK_OK;
            a.scale = (float)(1.0 / std::sqrt((double)d));
            a.eps = eps;
            a.n_rows = B;
            if (grouped) {
                const int G = nq / nkv;
                a.chunk_tokens = w.pf_chunk_tokens;
                a.max_chunks = w.pf_max_chunks;
                const dim3 grid(nkv, w.pf_max_chunks, (B + 16 / G - 1) / (16 / G));
                s = (d == 128) ? launch_prefill_attention_d<128>(a, G, grid, st)
                               : launch_prefill_attention_d<64>(a, G, grid, st);
            } else {
                a.plan = plan;
                const dim3 grid = plan ? dim3(nkv, B * w.max_chunks) : dim3(w.max_chunks, nkv, B);
                const bool use_mfma = w.attn_mfma;
                const int G = nq / nkv;
                if (plan)
                    s = (d == 128) ? launch_attention_d<128, true>(a, G, grid, use_mfma, w.attn_light, st)
                                   : launch_attention_d<64, true>(a, G, grid, use_mfma, w.attn_light, st);
                else
                    s = (d == 128) ? launch_attention_d<128, false>(a, G, grid, use_mfma, w.attn_light, st)
                                   : launch_attention_d<64, false>(a, G, grid, use_mfma, w.attn_light, st);
            }
            if (s != DK_OK) return s;
        }
        // x += W_o * attn
        if (batched) {
            dk::GemmArgs g{};
            g.W = u16(L.w_o);
            g.N = H;
            g.K = nq * d;
            g.B = B;
            g.q4 = model->q4;
            g.pack = w.pack_a;
            g.kpart = kpart;
            g.ktickets = ktickets;
            g.xhi = ahi;
            g.xlo = alo;
            g.xres = x;
            g.gain_next = u16(L.g_mlp);
            g.ohi = xhi;
            g.olo = xlo;
            g.ox3 = x3;
            g.ssq_out = ssq;
            if ((s = launch_gemm<dk::GEPI_RESID, false>(g, w.Bp, st)) != DK_OK) return s;
        } else {
            dk::GemvArgs g{};
            g.W = u16(L.w_o);
            g.x = attn;
            g.y = x;
            g.resid = x;
            g.N = H;
            g.K = nq * d;
            if (w.defer_merge) {
                g.part = part;
                g.seq_lens = d_seq_lens;
                g.chunk_tokens = w.chunk_tokens;
                g.max_chunks = w.max_chunks;
                g.max_blocks = max_blocks;
                g.group = nq / nkv;
                g.d = d;
                g.nkv = nkv;
                s = launch_gemv<dk::EPI_RESID, false, true>(g, B, st);
            } else {
                s = launch_gemv<dk::EPI_RESID, false>(g, B, st);
            }
            if (s != DK_OK) return s;
        }
        // act = silu(W_gate * h) * (W_up * h), h = rmsnorm(x);  x += W_down * act
        const uint16_t *gain_after = (l + 1 < c.n_layers) ? u16(model->layers[(size_t)l + 1].g_attn)
                                                           : u16(model->g_final);
        if (batched && c.n_experts > 0) {
            int *topk_idx = reinterpret_cast<int *>(ws + w.topk_idx) + (size_t)l * B * c.top_k;
            float *topk_w = reinterpret_cast<float *>(ws + w.topk_w);
            float *rinv = reinterpret_cast<float *>(ws + w.rinv);
            float *yexp = reinterpret_cast<float *>(ws + w.yexp);
            dk::RouterArgs r{};
            r.x = x;
            r.gain = u16(L.g_mlp);
            r.w_router = u16(L.w_router);
            r.eps = eps;
            r.H = H;
            r.E = c.n_experts;
            r.top_k = c.top_k;
            r.logits = reinterpret_cast<float *>(ws + w.rlogits);
            r.topk_idx = topk_idx;
            r.topk_w = topk_w;
            r.rinv = rinv;
            r.B = B;
            r.exp_cnt = reinterpret_cast<int *>(ws + w.exp_cnt);
            r.exp_list = reinterpret_cast<int *>(ws + w.exp_list);
            DK_LAUNCH(DK_K_MOE_ROUTER, dk::moe_router_logits_kernel, dim3((c.n_experts + 7) / 8, B), dim3(256),
                      0, st, r);
            DK_LAUNCH(DK_K_MOE_ROUTER, dk::moe_router_select_kernel, dim3(B), dim3(64), 0, st, r);
            DK_HIP(hipGetLastError());
            if (l + 1 == c.n_layers && kv_only) return DK_OK;
            dk::ExpertArgs up{};
            up.w_a = u16(L.w_gate);
            up.w_b = u16(L.w_up);
            up.N = c.expert_ffn;
            up.K = H;
            up.n_experts = c.n_experts;
            up.B = B;
            up.top_k = c.top_k;
            up.exp_cnt = r.exp_cnt;
            up.exp_list = r.exp_list;
            up.xhi = xhi;
            up.xlo = xlo;
            up.rinv = rinv;
            up.ohi = fhi;
            up.olo = flo;
            // K a multiple of 128 and at least one k-step per wave: the restructured kernel
            if (model->q4) {   // shapes checked by dk_create_model_q4
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_fast_kernel<true, 4, 1, 2, true>),
                          dim3((c.expert_ffn + 15) / 16, c.n_experts), dim3(256), 0, st, up);
            } else if (H % 128 == 0 && H / 128 >= 4) {
                // measured at the 30B-A3B shape: small blocks (4 waves, one 16-row tile, two
                // k-steps per round) so that many are resident per compute unit
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_fast_kernel<true, 4, 1, 2>),
                          dim3((c.expert_ffn + 15) / 16, c.n_experts), dim3(256), 0, st, up);
            } else {
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_kernel<true, 8>),
                          dim3((c.expert_ffn + 15) / 16, c.n_experts), dim3(512), 0, st, up);
            }
            DK_HIP(hipGetLastError());
            dk::ExpertArgs dn{};
            dn.w_a = u16(L.w_down);
            dn.N = H;
            dn.K = c.expert_ffn;
            dn.n_experts = c.n_experts;
            dn.B = B;
            dn.top_k = c.top_k;
            dn.exp_cnt = r.exp_cnt;
            dn.exp_list = r.exp_list;
            dn.xhi = fhi;
            dn.xlo = flo;
            dn.y = yexp;
            if (model->q4 && c.expert_ffn % 768 == 0) {
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_fast_kernel<false, 3, 2, 2, true>), dim3((H + 31) / 32, c.n_experts),
                          dim3(192), 0, st, dn);
            } else if (model->q4) {
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_fast_kernel<false, 4, 2, 1, true>), dim3((H + 31) / 32, c.n_experts),
                          dim3(256), 0, st, dn);
            } else if (c.expert_ffn % 768 == 0) {          // six k-steps (or a multiple): 3 waves x 2 per round
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_fast_kernel<false, 3, 2, 2>), dim3((H + 31) / 32, c.n_experts),
                          dim3(192), 0, st, dn);
            } else if (c.expert_ffn % 128 == 0 && c.expert_ffn / 128 >= 4) {
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_fast_kernel<false, 4, 2, 1>), dim3((H + 31) / 32, c.n_experts),
                          dim3(256), 0, st, dn);
            } else {
                DK_LAUNCH(DK_K_MOE_EXPERT, (dk::moe_expert_kernel<false, 4>), dim3((H + 15) / 16, c.n_experts),
                          dim3(256), 0, st, dn);
            }
            DK_HIP(hipGetLastError());
            dk::MoeCombineArgs cb{};
            cb.x = x;
            cb.y = yexp;
            cb.topk_w = topk_w;
            cb.gain_next = gain_after;
            cb.xhi = xhi;
            cb.xlo = xlo;
            cb.ssq_out = ssq;
            cb.H = H;
            cb.top_k = c.top_k;
            DK_LAUNCH(DK_K_MOE_COMBINE, dk::moe_combine_kernel, dim3((H + 1023) / 1024, B), dim3(256), 0, st, cb);
            DK_HIP(hipGetLastError());
        } else if (batched) {
            dk::GemmArgs g{};
            g.W = u16(L.w_gate);
            g.W2 = u16(L.w_up);
            g.N = c.ffn;
            g.K = H;
            g.B = B;
            g.q4 = model->q4;
            g.spread = !prefill;
            g.pack = w.pack_x;
            g.kpart = kpart;
            g.ktickets = ktickets;
            g.xhi = xhi;
            g.xlo = xlo;
            g.ssq_in = ssq;
            g.n_part = ssq_tiles;
            g.eps = eps;
            g.ohi = fhi;
            g.olo = flo;
            g.ox3 = f3;
            if ((s = launch_gemm<dk::GEPI_SWIGLU, true>(g, w.Bp, st)) != DK_OK) return s;
            dk::GemmArgs h{};
            h.W = u16(L.w_down);
            h.N = H;
            h.K = c.ffn;
            h.B = B;
            h.q4 = model->q4;
            h.pack = w.pack_f;
            h.kpart = kpart;
            h.ktickets = ktickets;
            h.xhi = fhi;
            h.xlo = flo;
            h.xres = x;
            h.gain_next = gain_after;
            h.ohi = xhi;
            h.olo = xlo;
            h.ox3 = x3;
            h.ssq_out = ssq;
            if ((s = launch_gemm<dk::GEPI_RESID, false>(h, w.Bp, st)) != DK_OK) return s;
        } else {
            dk::GemvArgs g{};
            g.W = u16(L.w_gate);
            g.W2 = u16(L.w_up);
            g.x = x;
            g.gain = u16(L.g_mlp);
            g.eps = eps;
            g.y = act;
            g.N = c.ffn;
            g.K = H;
            if ((s = launch_gemv<dk::EPI_SWIGLU, true>(g, B, st)) != DK_OK) return s;
            dk::GemvArgs h{};
            h.W = u16(L.w_down);
            h.x = act;
            h.y = x;
            h.resid = x;
            h.N = H;
            h.K = c.ffn;
            if ((s = launch_gemv<dk::EPI_RESID, false>(h, B, st)) != DK_OK) return s;
        }
    }

    if (d_next_tokens == nullptr) return fail(DK_E_INVALID_ARG, "NULL argument");
    // logits = W_lm * rmsnorm(x); greedy token
    if (batched) {
        dk::GemmArgs g{};
        g.W = u16(model->lm_head);
        g.N = c.vocab;
        g.K = H;
        g.B = B;
        g.q4 = model->q4;
        g.pack = w.pack_x;
        g.kpart = kpart;
        g.ktickets = ktickets;
        g.xhi = xhi;
        g.xlo = xlo;
        g.ssq_in = ssq;
        g.n_part = c.n_experts > 0 ? (H + 1023) / 1024 : ssq_tiles;
        g.eps = eps;
        g.y = d_logits;
        g.pmax_val = pmax_val;
        g.pmax_idx = pmax_idx;
        if ((s = launch_gemm<dk::GEPI_STORE, true>(g, w.Bp, st)) != DK_OK) return s;
    } else {
        dk::GemvArgs g{};
        g.W = u16(model->lm_head);
        g.x = x;
        g.gain = u16(model->g_final);
        g.eps = eps;
        g.N = c.vocab;
        g.K = H;
        g.pmax_val = pmax_val;
        g.pmax_idx = pmax_idx;
        g.tiles = kLmTiles;
        g.y = d_logits;   // may be null: then only the running maxima are kept
        if ((s = launch_gemv<dk::EPI_STORE, true>(g, B, st)) != DK_OK) return s;
    }
    dk::ArgmaxArgs am{pmax_val, pmax_idx, w.lm_blocks, d_next_tokens, d_tokens, d_seq_lens,
                      (flags & DK_STEP_ADVANCE) ? 1 : 0};
    DK_LAUNCH(DK_K_ARGMAX, dk::argmax_final_kernel, dim3(B), dim3(1024), 0, st, am);
    DK_HIP(hipGetLastError());
    return DK_OK;
}

dk_status dk_debug_set_wait_limit(dk_model *model, int32_t polls)
{
    if (!model) return fail(DK_E_INVALID_ARG, "model is NULL");
    if (polls < 0) return fail(DK_E_INVALID_ARG, "polls %d", polls);
    model->fused_spin_limit = polls > 0 ? polls : dk::kFusedSpinLimit;
    return DK_OK;
}

dk_status dk_debug_set_stage_stamps(dk_model *model, int32_t layer, void *d_stamps, size_t stamps_bytes)
{
    if (!model) return fail(DK_E_INVALID_ARG, "model is NULL");
    if (d_stamps == nullptr) {
        model->fused_stamps = nullptr;
        return DK_OK;
    }
    if (layer < 0 || layer >= model->cfg.n_layers) return fail(DK_E_INVALID_ARG, "layer %d of %d", layer, model->cfg.n_layers);
    const size_t need = (size_t)fused_blocks() * dk::kFusedStamps * sizeof(long long);
    if (stamps_bytes < need || (uintptr_t)d_stamps % 8)
        return fail(DK_E_INVALID_ARG, "stamp buffer of %zu bytes (%zu needed, 8-byte aligned)", stamps_bytes, need);
    model->fused_stamps = static_cast<long long *>(d_stamps);
    model->fused_stamp_layer = layer;
    return DK_OK;
}

dk_status dk_workspace_reset(dk_model *model)
{
    if (!model) return fail(DK_E_INVALID_ARG, "model is NULL");
    model->fused_ws = nullptr;
    model->fused_ws_bytes = 0;
    return DK_OK;
}

dk_status dk_fused_status(const dk_model *model, const void *d_workspace, uint32_t *out, void *hip_stream)
{
    if (!model || !d_workspace || !out) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (model->fused_ws != d_workspace)
        return fail(DK_E_INVALID_ARG, "this workspace has not been used by a persistent step of the model");
    // the status words sit at the end of the workspace layout the last step used
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    DK_HIP(hipMemcpyAsync(out, static_cast<const char *>(d_workspace) + model->fused_ws_bytes - 256, 8,
                          hipMemcpyDeviceToHost, st));
    DK_HIP(hipStreamSynchronize(st));
    return DK_OK;
}

dk_status dk_step_routing(const dk_model *model, const void *d_workspace, int32_t B,
                          int32_t max_blocks, int32_t *h_out, void *hip_stream)
{
    if (!model || !d_workspace || !h_out) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (model->cfg.n_experts <= 0) return fail(DK_E_INVALID_ARG, "the model has no expert layers");
    if (B <= 0 || B > DK_MAX_BATCH || max_blocks <= 0) return fail(DK_E_INVALID_ARG, "B %d, max_blocks_per_seq %d", B, max_blocks);
    const Workspace w = carve(model->cfg, B, max_blocks, model->q4);
    const size_t bytes = (size_t)model->cfg.n_layers * B * model->cfg.top_k * 4;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    DK_HIP(hipMemcpyAsync(h_out, static_cast<const char *>(d_workspace) + w.topk_idx, bytes,
                          hipMemcpyDeviceToHost, st));
    DK_HIP(hipStreamSynchronize(st));
    return DK_OK;
}

dk_status dk_step_algorithmic_bytes(const dk_model *model, const dk_kv_pool *pool,
                                    const int32_t *bt, int32_t max_blocks, const int32_t *seq_lens,
                                    int32_t B, int32_t with_logits, const int32_t *distinct_experts,
                                    uint64_t *out_bytes)
{
    if (!model || !pool || !bt || !seq_lens || !out_bytes) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (B <= 0 || max_blocks <= 0) return fail(DK_E_INVALID_ARG, "B %d, max_blocks_per_seq %d", B, max_blocks);
    const dk_model_config &c = model->cfg;
    const uint64_t H = (uint64_t)c.hidden, d = (uint64_t)c.head_dim;
    const uint64_t qd = (uint64_t)c.n_q_heads * d, kvd = (uint64_t)c.n_kv_heads * d;
    uint64_t per_layer = H * qd + 2 * H * kvd + qd * H;   // q, k, v, o
    uint64_t bytes = 0;
    if (c.n_experts > 0) {
        if (!distinct_experts) return fail(DK_E_INVALID_ARG, "MoE model needs distinct_experts_per_layer");
        for (int l = 0; l < c.n_layers; l++) {
            const uint64_t ew = (uint64_t)distinct_experts[l] * 3 * H * (uint64_t)c.expert_ffn;
            bytes += model->q4 ? ew / 2 + ew / 64 * 4 : 2 * ew;
        }
        bytes += 2 * (uint64_t)c.n_layers * c.n_experts * H;   // routers (bf16 in either format)
    } else {
        per_layer += 3 * H * (uint64_t)c.ffn;
    }
    const uint64_t weights = (uint64_t)c.n_layers * per_layer + (uint64_t)c.vocab * H;
    if (model->q4) {
        // half a byte per weight plus a bf16 scale and bias per 64 weights; norm gains, routers and
        // the embedding aside, every matrix of a 4-bit model is in that format
        bytes += weights / 2 + weights / 64 * 4;
    } else {
        bytes += 2 * weights;
    }
    // live KV: every distinct (block, slot) once, including this step's token
    std::set<int64_t> slots;
    for (int32_t b = 0; b < B; b++) {
        const int32_t T = seq_lens[b];
        if (T < 0 || T / pool->block_size >= max_blocks)
            return fail(DK_E_INVALID_ARG, "row %d: seq_len %d does not fit the table", b, T);
        for (int32_t t = 0; t <= T; t++) {
            const int32_t id = bt[(size_t)b * max_blocks + t / pool->block_size];
            if (id < 0 || id >= pool->num_blocks)
                return fail(DK_E_BAD_BLOCK, "row %d: block %d out of range", b, id);
            slots.insert((int64_t)id * pool->block_size + t % pool->block_size);
        }
    }
    bytes += (uint64_t)slots.size() * (uint64_t)c.n_layers * 2 * kvd * 2;
    bytes += (uint64_t)B * H * 2;                                   // embedding rows
    if (with_logits) bytes += (uint64_t)B * (uint64_t)c.vocab * 4;  // logits written
    *out_bytes = bytes;
    return DK_OK;
}

dk_status dk_read_stream(const void *d_buf, size_t bytes, void *d_sink, void *hip_stream)
{
    if (!d_buf || !d_sink) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (bytes == 0 || bytes % 16 || (uintptr_t)d_buf % 16) return fail(DK_E_INVALID_ARG, "bytes %zu (a positive multiple of 16, 16-byte aligned)", bytes);
    // one block per compute unit, looping: the shape that read fastest in sweeps of 256..65536 blocks of
    // 256..1024 threads, grid-strided or one contiguous chunk per block (6.6 TB/s against 5.2-6.3)
    int dev = 0, cus = 0;
    DK_HIP(hipGetDevice(&dev));
    DK_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    hipLaunchKernelGGL(read_stream_kernel, dim3(cus > 0 ? cus : 256), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<const uint4 *>(d_buf), bytes / 16, static_cast<uint32_t *>(d_sink));
    DK_HIP(hipGetLastError());
    return DK_OK;
}

dk_status dk_gemm_plan_query(int32_t epilogue, int32_t N, int32_t K, int32_t B, int32_t four_bit,
                             int32_t compute_units, int32_t *out_waves, int32_t *out_slices,
                             double *out_estimate_us)
{
    if (!out_waves || !out_slices || !out_estimate_us) return fail(DK_E_INVALID_ARG, "NULL argument");
    if (epilogue < 0 || epilogue > 2 || N < 1 || K < 1 || B <= kMaxGemvBatch || B > DK_MAX_BATCH || compute_units < 0)
        return fail(DK_E_INVALID_ARG, "epilogue %d, N %d, K %d, B %d, compute units %d", epilogue, N, K, B, compute_units);
    const int Bp = (B + 15) / 16 * 16;
    const int cus = compute_units ? compute_units : device_cus();
    const GemmPlan p = dkplan::gemm_plan(epilogue, N, K, Bp, four_bit != 0, B <= kPackRows2 && K % 128 == 0, cus, out_estimate_us);
    *out_waves = dkplan::shared_waves(epilogue, N, Bp / 16, p, cus);
    *out_slices = p.slices;
    return DK_OK;
}

}  // extern "C"

// continuous-batching scheduler and prefix cache on top of the entry points above
#include "dk_engine.hip.h"
