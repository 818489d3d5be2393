// Host side of the C ABI declared in include/saber.h: validation, the device data layout, and the
// per-iteration launch sequence of Alg. 1.  Every step of the path runs in the kernels of
// saber_kernels.hpp; nothing here computes counts or samples on the CPU.
#include "saber_kernels.hpp"
#include "saber_ablation.hpp"
#include "../../include/saber.h"
#include "../../include/saber_measure.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <system_error>
#include <thread>
#include <vector>

#include <rocprim/rocprim.hpp>

using namespace saber;

// ------------------------------------------------------------------------------------------------
// errors
// ------------------------------------------------------------------------------------------------
static thread_local char g_err[512] = "";
static int fail(int code, const char *fmt, ...) {
    // the runtime keeps the thread's last error until it is asked for: left there, it would be taken for the next launch's
    if (code == SABER_ENOMEM || code == SABER_EDEVICE) (void)hipGetLastError();
    va_list ap; va_start(ap, fmt); vsnprintf(g_err, sizeof(g_err), fmt, ap); va_end(ap);
    return code;
}
#define HIP_TRY(expr)                                                                                     \
    do {                                                                                                  \
        hipError_t e_ = (expr);                                                                           \
        if (e_ != hipSuccess)                                                                             \
            return fail(e_ == hipErrorOutOfMemory ? SABER_ENOMEM : SABER_EDEVICE, "%s failed: %s (%s:%d)", \
                        #expr, hipGetErrorString(e_), __FILE__, __LINE__);                                \
    } while (0)
#define SABER_TRY(expr) do { int rc_ = (expr); if (rc_ != SABER_OK) return rc_; } while (0)

extern "C" const char *saber_last_error(void) { return g_err; }

// ------------------------------------------------------------------------------------------------
// device memory
// ------------------------------------------------------------------------------------------------
// Work space of the log-likelihood reduction: the per-tile sums of one chunk, then kLlTail doubles - the workgroup sums
// of one reduction pass, the running total over chunks, the normaliser and the result.
constexpr size_t kLlTail = (size_t)kReduceBlocks + 3;
struct LlScratch { double *tile_part, *block_part, *acc, *norm, *result; };
static LlScratch ll_scratch(double *base, size_t max_tiles) {
    LlScratch w;
    w.tile_part = base; w.block_part = base + max_tiles; w.acc = w.block_part + kReduceBlocks; w.norm = w.acc + 1; w.result = w.norm + 1;
    return w;
}

// Where device memory and the compute stream come from (saber_set_hooks).  A context keeps the hooks it was created
// with, so its memory goes back through the deallocator that matches its allocator.
struct Hooks {
    void *(*alloc)(size_t) = nullptr;
    void (*dealloc)(void *) = nullptr;
    hipStream_t stream = nullptr;
    bool have_stream = false;
};
static Hooks g_hooks;

static int hook_alloc(const Hooks &h, void **p, size_t bytes) {
    *p = nullptr;
    bytes = std::max<size_t>(bytes, 1);
    if (h.alloc) {
        *p = h.alloc(bytes);
        if (!*p) return fail(SABER_ENOMEM, "the caller's allocator returned no memory for %zu bytes", bytes);
        if (reinterpret_cast<uintptr_t>(*p) & 255u) {
            void *q = *p; *p = nullptr;
            if (h.dealloc) h.dealloc(q);
            return fail(SABER_EINVAL, "the caller's allocator returned memory that is not 256-byte aligned");
        }
        return SABER_OK;
    }
    HIP_TRY(hipMalloc(p, bytes));
    return SABER_OK;
}
static void hook_free(const Hooks &h, void *p) {
    if (!p) return;
    if (h.alloc) { if (h.dealloc) h.dealloc(p); }
    else (void)hipFree(p);
}
template <typename T>
static int dev_alloc(const Hooks &h, T **p, size_t n) { return hook_alloc(h, (void **)p, std::max<size_t>(n, 1) * sizeof(T)); }
static void dev_free(const Hooks &h, void *p) { hook_free(h, p); }

// ------------------------------------------------------------------------------------------------
// context
// ------------------------------------------------------------------------------------------------
// Tiles of a chunk that are launched together: `count` tiles from the chunk's tile `first` on, the first `n_dense` of them of
// words with dense rows, workgroups of `block` threads
struct TileClass { int64_t first, count, n_dense; int block; };

struct Chunk {
    int64_t d0 = 0, d1 = 0;   // document range
    int64_t t0 = 0, ntok = 0; // canonical token range [t0, t0+ntok)
    int64_t tile0 = 0, ntiles = 0, words_present = 0;
    // tiles of the chunk: first those of words with dense B rows, then those of light words (sparse B rows), each
    // group sorted by decreasing size and cut into classes by size
    std::vector<TileClass> classes;
    // the chunk's documents inside the (ascending) lists of short and of long documents
    int64_t short0 = 0, nshort = 0, long0 = 0, nlong = 0;
    // the rows of A of the chunk's documents: first row and extent, in units of 32 entries (128 bytes)
    int64_t row_unit0 = 0, row_units = 0;
};

constexpr int kMaxSlots = 8;
constexpr int kPullSlots = 12, kPullThreads = 8;      // see pull()
constexpr int64_t kPullPiece = 1 << 20;               // bytes
// Bytes written for the caller up to which plain copies do, and from which on threads are worth their start and the large
// staging, or if that is there already (`next`) their start: for assignments, which are only widened; entries of A, which
// are taken apart; rows of B, copied or filled in.
struct PullBy { int64_t few, many, next; };
constexpr PullBy kPullZ = {4 << 20, 8 << 20, 8 << 20}, kPullEntries = {1 << 20, 8 << 20, 1 << 20}, kPullRows = {4 << 20, 8 << 20, 1 << 20};
// Pinned staging of results and the events of its slots, made by the first call that needs them.
struct Staging { char *buf = nullptr; size_t bytes = 0; bool pinned = false; hipEvent_t ev[kPullSlots] = {}; };

constexpr int kMaxTimedIters = 32;
constexpr int kCtr = 8;   // device counters per timed iteration
enum { EV_BEGIN = 0, EV_SAMPLE, EV_DZ, EV_CK, EV_PHI, EV_PER_ITER };

struct saber_ctx {
    Hooks hooks;                      // allocator and stream in force when the context was created
    bool own_stream = false;
    int device = 0;                   // the HIP device the context lives on
    int64_t D = 0, T = 0;
    int32_t V = 0, K = 0, Kpad = 0, n3 = 0, n3pad = 0, nwords = 0;
    float alpha = 0, beta = 0, vbeta = 0;
    uint64_t seed = 0;
    uint32_t iter = 0, topic_bits = 0, count_bits = 0;   // (a packed entry: the topic above the count)
    bool z16 = false, staged = false, b16 = false;
    int pack = PACK_ANY;              // what a kernel may take for granted of the entries of this context's rows of A
    bool slots = false;               // sampling wavefronts have a part of LDS of their own (estep_kernel, SLOTS)
    bool overlay = false;             // rows do not fit LDS: light words are read from memory with marks in LDS (Overlay)
    bool auto_light_block = false;    // neither workgroup size was given: those of light words' tiles follow the tile
    int lds_per_cu = 64 * 1024, cus = 256;
    saber_options opt{};
    int32_t tile_tokens_asked = 0;    // the caller's tile_tokens (0: automatic), before the default was filled in
    int64_t max_doc_len = 0;
    hipStream_t stream = nullptr;
    // device arrays
    void *z = nullptr;                // [T] uint16 or int32, canonical (document) order
    int32_t *tok_doc = nullptr;       // [T] word-major inside every chunk
    uint32_t *tok_t = nullptr;        // [T]
    Tile *tiles = nullptr;
    uint2 *docrec = nullptr;          // [D]
    uint32_t *cd_ent = nullptr;       // [cd_cap]
    int64_t cd_cap = 0;
    int64_t *doc_ptr = nullptr;       // [D+1]
    int32_t *short_docs = nullptr, *long_docs = nullptr;
    int64_t n_short = 0, n_long = 0;
    // words: V_dense keep dense rows of B and Bhat (row V_dense is an all-zero row that yields the base vector);
    // V_light keep B sparse, like the rows of A
    int32_t V_dense = 0, V_light = 0;
    int32_t *row_word = nullptr;      // [V_dense+1] word of each dense row (the zero row maps to word index V)
    int32_t *light_words = nullptr;   // [V_light] word of each light row
    int32_t *light_short = nullptr, *light_long = nullptr;   // light rows by token count, for the count launches
    int64_t n_light_short = 0, n_light_long = 0;
    int32_t n_light_wide = 0;         // light rows of words with more than kWideWord tokens: they have the first numbers
    int64_t *light_tok_ptr = nullptr; // [V_light+1] positions of the light words' tokens in z_wm
    uint2 *wrec = nullptr;            // [V_light] {row start / 32, non-zeros}
    uint32_t *lw_ent = nullptr;       // packed rows of B of the light words
    float *lw_phi = nullptr;          // Bhat of each such entry
    void *z_wm = nullptr;             // [T] word-major assignments: the light words' tokens first, then the dense rows' ones
    int64_t T_light = 0, lw_cap = 0;
    VzItem *vz_items = nullptr;       // slabs of the dense-row words' segments of z_wm, those of the longest rows first
    int64_t n_vz_items = 0, n_vz_long = 0;   // all; those of rows that are not counted where they are normalised
    PhiRow *phi_rows = nullptr;       // [V_dense+1] the dense rows as phi_row() takes them
    bool joined = false;              // the M-step takes two launches (see launch_joined_mstep)
    std::vector<int32_t> h_word_row;  // host: word -> dense row (>= 0) or -(light row) - 1
    // A context built on a trained model (held-out documents): it borrows the model's word classes, Bhat, tree
    // levels and sparse rows, owns only its own tokens, z and rows of A, and never rebuilds B.
    const saber_ctx *parent = nullptr;
    bool no_state = false;            // no assignments of its own (tokens that are only scored)
    int32_t *cwk = nullptr;           // [V_dense+1][Kpad]
    unsigned long long *ck = nullptr, *ck_acc = nullptr; // [K] topic totals; their accumulators, zero outside the M-step, and a
                                                         // ticket counter behind them, likewise
    bool acc_used = true;             // cwk or ck_acc may hold counts: set before any are added, cleared once what empties them is queued
    float *denom = nullptr;           // [K] denominators of Eq. 2
    float *phi = nullptr, *l3 = nullptr, *sumphi = nullptr;
    double *l3_64 = nullptr;          // [V][n3]
    uint32_t *doc_words = nullptr;    // [D] distinct words of the document
    unsigned long long *dense_slots = nullptr; // [kMaxTimedIters][kDenseSlots] dense-branch tokens, spread over slots
    unsigned long long *counters = nullptr; // [kMaxTimedIters][kCtr]: dense-branch tokens, nnz(A), sum K_d L_d, sum K_d U_d,
                                            // non-zeros of the sparse rows of B
    // log-likelihood reduction: [max tiles per chunk] per-tile sums, then kLlTail doubles (LlScratch below)
    double *ll_partial = nullptr;
    std::vector<Chunk> chunks;
    int64_t total_tiles = 0, max_chunk_tiles = 0;
    // measurement
    hipEvent_t ev[kMaxTimedIters * EV_PER_ITER] = {};
    bool have_events = false;
    saber_stats stats{};
    Staging staging;                  // device -> host results, see pull()
    void *work = nullptr;             // device memory of the inspection calls, see WorkSpace
    size_t work_bytes = 0;
    std::vector<int64_t> doc_len;     // host copy of the document lengths (statistics only)
    // Host streaming (Sec. 3.1.2), n_slots > 0: tok_t lives in pinned host memory; a chunk's part of it is copied
    // into one of n_slots device buffers for the chunk's pass (4 bytes per token and iteration over the host link).
    // The rest is derived or kept on the device: the chunk's tok_doc follows, on a third stream, from one look-up per token in
    // doc_blocks (16 bytes per 64 canonical tokens: where documents start); its assignments in document order exist only in the
    // buffer, between the sampling kernel that writes them and the CountByDZ that turns them into rows of A, and
    // are re-created from the word-major copy when asked for; z_wm (2 bytes per token) and the rows of A are
    // resident.  Copies run on a stream of their own; the three are ordered with three events per buffer.
    int n_slots = 0, next_slot = 0;
    int64_t slot_tokens = 0;
    uint32_t *h_tok_t = nullptr;
    uint4 *doc_blocks = nullptr;      // [ceil(T/64)] see expand_tok_doc_kernel
    int32_t *ne_doc = nullptr;        // [non-empty documents] their numbers; null when no document is empty
    int32_t *slot_tok_doc[kMaxSlots] = {}; uint32_t *slot_tok_t[kMaxSlots] = {}; void *slot_z[kMaxSlots] = {};
    hipStream_t s_in = nullptr, s_docs = nullptr;   // copies; the expansion of their tok_doc
    hipEvent_t ev_copied[kMaxSlots] = {}, ev_loaded[kMaxSlots] = {}, ev_done[kMaxSlots] = {};
    bool slot_used[kMaxSlots] = {};   // ev_done says when its last user's kernels are done
    bool slot_open[kMaxSlots] = {};   // loaded, and ev_done not recorded since
    // ablation variants (saber_options.ablation): document-order sampling needs the words in canonical order and
    // the word -> row map; the sort-based rebuild of A needs key buffers and the sort's work space
    int32_t *word_ids_d = nullptr, *word_row_d = nullptr;
    uint64_t *sort_keys = nullptr, *sort_keys_out = nullptr;
    uint32_t *sort_rank = nullptr;
    void *sort_tmp = nullptr;
    size_t sort_tmp_bytes = 0;
    unsigned sort_end_bit = 0;
    uint2 *alias_table = nullptr;     // [V_dense][K] {prob bits, alias} when the dense term is drawn from alias tables
};

static inline int grid_for(int64_t n, int block, int cap = 65535 * 16) {
    int64_t g = (n + block - 1) / block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

// A grid has at most 2^32 - 1 threads in a dimension: what a launch of workgroups of `block` threads can take.  A longer
// list of work is launched by pieces.
static inline int64_t most_blocks(int block) { return 0xffffffffll / block; }

extern "C" int saber_set_hooks(void *(*alloc)(size_t), void (*dealloc)(void *), void *hip_stream) {
    if ((alloc == nullptr) != (dealloc == nullptr))
        return fail(SABER_EINVAL, "saber_set_hooks: alloc and dealloc must be given together");
    g_hooks.alloc = alloc; g_hooks.dealloc = dealloc;
    g_hooks.stream = reinterpret_cast<hipStream_t>(hip_stream); g_hooks.have_stream = hip_stream != nullptr;
    return SABER_OK;
}

extern "C" void saber_options_default(saber_options *opt) {
    if (!opt) return;
    memset(opt, 0, sizeof(*opt));
    opt->n_chunks = 0; opt->block_threads = 0; opt->tile_tokens = 0; opt->stage_phi = 1; opt->profile = 0;
    opt->quarter_row_entries = 64; opt->half_row_entries = 128;
    opt->long_doc_tokens = 512; opt->dz_lds_entries = 2048; opt->stage_min_tokens = 0; opt->light_block_threads = 0; opt->light_word_tokens = 0;
}

extern "C" void saber_free(saber_ctx *c) {
    if (!c) return;
    if (c->stream) (void)hipStreamSynchronize(c->stream);
    auto release = [c](void *p) { dev_free(c->hooks, p); };
    release(c->z); release(c->tok_doc); release(c->tok_t); release(c->tiles); release(c->docrec);
    release(c->cd_ent); release(c->doc_ptr); release(c->short_docs); release(c->long_docs);
    release(c->doc_words); release(c->counters); release(c->dense_slots); release(c->ll_partial); release(c->z_wm);
    if (!c->parent) {   // the model's arrays belong to the model
        release(c->cwk); release(c->ck); release(c->ck_acc); release(c->denom); release(c->phi); release(c->l3_64); release(c->l3);
        release(c->sumphi); release(c->row_word); release(c->light_words); release(c->light_short);
        release(c->light_long); release(c->light_tok_ptr); release(c->wrec); release(c->lw_ent); release(c->lw_phi);
        release(c->vz_items); release(c->phi_rows);
    }
    if (c->have_events) for (auto &e : c->ev) if (e) (void)hipEventDestroy(e);
    for (hipStream_t s : {c->s_in, c->s_docs}) if (s) { (void)hipStreamSynchronize(s); (void)hipStreamDestroy(s); }
    for (int s = 0; s < kMaxSlots; s++) {
        release(c->slot_tok_doc[s]); release(c->slot_tok_t[s]); release(c->slot_z[s]);
        if (c->ev_copied[s]) (void)hipEventDestroy(c->ev_copied[s]);
        if (c->ev_loaded[s]) (void)hipEventDestroy(c->ev_loaded[s]);
        if (c->ev_done[s]) (void)hipEventDestroy(c->ev_done[s]);
    }
    release(c->doc_blocks); release(c->ne_doc); release(c->work);
    release(c->word_ids_d); release(c->word_row_d); release(c->sort_keys); release(c->sort_keys_out);
    release(c->sort_rank); release(c->sort_tmp); release(c->alias_table);
    if (c->h_tok_t) (void)hipHostFree(c->h_tok_t);
    if (c->staging.buf) { if (c->staging.pinned) (void)hipHostFree(c->staging.buf); else free(c->staging.buf); }
    for (auto &e : c->staging.ev) if (e) (void)hipEventDestroy(e);
    if (c->stream && c->own_stream) (void)hipStreamDestroy(c->stream);
    delete c;
}

// ------------------------------------------------------------------------------------------------
// launch helpers
// ------------------------------------------------------------------------------------------------
// The assignments of a chunk in canonical order: the resident array, which holds all tokens (`first` = 0: its first
// element is token 0), or the streaming buffer that holds the chunk (`first` = the chunk's first token).
struct ZView { void *z; int64_t first; };
static ZView z_view(const saber_ctx *c, const Chunk &ch, int slot) {
    return slot < 0 ? ZView{c->z, 0} : ZView{c->slot_z[slot], ch.t0};
}

// The rows of A the sampling kernel reads for the documents of chunk `ch` of context `theta`: all of them sit behind
// one buffer descriptor and are addressed by 32-bit byte offsets (lay_out() keeps every chunk's rows below 4 GB).
static void set_rows(EStepParams &p, const saber_ctx *theta, const Chunk &ch) {
    p.docrec = theta->docrec;
    p.cd_rows = theta->cd_ent + (size_t)ch.row_unit0 * 32u;
    p.row_unit0 = (uint32_t)ch.row_unit0;
    p.rows_bytes = (uint32_t)((uint64_t)ch.row_units * 128u);
    p.quarter_row_bytes = 4u * (uint32_t)theta->opt.quarter_row_entries; p.half_row_bytes = 4u * (uint32_t)theta->opt.half_row_entries;
}

// everything but the rows of A, which launch_estep() adds
static EStepParams make_params(saber_ctx *c, const Chunk &ch, int slot = -1) {
    EStepParams p{};
    p.tiles = c->tiles + ch.tile0;
    if (slot < 0) { p.tok_doc = c->tok_doc + ch.t0; p.tok_t = c->tok_t + ch.t0; }
    else { p.tok_doc = c->slot_tok_doc[slot]; p.tok_t = c->slot_tok_t[slot]; }
    p.phi = c->phi; p.l3 = c->l3; p.l3_64 = c->l3_64; p.sumphi = c->sumphi;
    const ZView zv = z_view(c, ch, slot);
    p.z = zv.z; p.z_rel = ch.t0 - zv.first;
    p.base = c->phi + (size_t)c->V_dense * (size_t)c->Kpad;
    p.wrec = c->wrec; p.lw_ent = c->lw_ent; p.lw_phi = c->lw_phi; p.z_wm = c->z_wm;
    p.alias_table = c->alias_table;
    p.t_base = ch.t0; p.K = c->K; p.Kpad = c->Kpad; p.n3 = c->n3; p.n3pad = c->n3pad;
    p.count_bits = c->count_bits; p.alpha = c->alpha;
    p.seed_lo = (uint32_t)c->seed; p.seed_hi = (uint32_t)(c->seed >> 32); p.iter = c->iter;
    return p;
}

// LDS of a staged sampling workgroup's row: the Bhat row (K rounded to 4 floats) and the tree level (n3 rounded to 4)
static size_t estep_row_bytes(const saber_ctx *c) {
    return ((size_t)((c->K + 3) & ~3) + (size_t)((c->n3 + 3) & ~3)) * sizeof(float);
}
// dynamic LDS of a sampling workgroup: the row when staged, 16 bytes of control words, in log-likelihood mode
// one double per wavefront, and kSlotBytes for each where they are used
static size_t estep_lds_bytes(const saber_ctx *c, int mode, int block) {
    if (c->overlay) return 16 + 16 * sizeof(double) + (size_t)c->nwords * sizeof(uint2);
    return (c->staged ? estep_row_bytes(c) : 0) + 16 + (mode == MODE_LOGLIK ? 16 * sizeof(double) : 0) +
           (c->slots && mode == MODE_SAMPLE ? (size_t)(block / 64) * kSlotBytes : 0);
}

// a workgroup may use more than the default 64 KB of LDS (up to the CU's 160 KB) once the kernel has been told so
template <typename Kern>
static void launch_with_lds(Kern kern, dim3 grid, dim3 block, size_t lds, hipStream_t stream, const EStepParams &p) {
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, grid, block, lds, stream, p);
}

template <int MODE, bool STAGED, typename ZT>
static void launch_estep_packed(saber_ctx *c, int pack, dim3 grid, dim3 block, size_t lds, const EStepParams &p) {
    if (MODE == MODE_SAMPLE && STAGED && sizeof(ZT) == 2 && c->slots)
        launch_with_lds(estep_kernel<MODE_SAMPLE, true, uint16_t, PACK_16_14, true>, grid, block, lds, c->stream, p);
    else if (STAGED && pack == PACK_16_14) launch_with_lds(estep_kernel<MODE, STAGED, ZT, STAGED ? PACK_16_14 : PACK_16>, grid, block, lds, c->stream, p);
    else if (pack != PACK_ANY) launch_with_lds(estep_kernel<MODE, STAGED, ZT, PACK_16>, grid, block, lds, c->stream, p);
    else launch_with_lds(estep_kernel<MODE, STAGED, ZT, PACK_ANY>, grid, block, lds, c->stream, p);
}

// The staged 16/16 sampler addresses its Bhat row from LDS address 0: its kernels must have no static LDS in
// front of the dynamic part.
template <typename F>
static int static_lds_is_zero(F kernel) {
    hipFuncAttributes a;
    HIP_TRY(hipFuncGetAttributes(&a, reinterpret_cast<const void *>(kernel)));
    if (a.sharedSizeBytes != 0) return fail(SABER_EDEVICE, "sampling kernel built with %zu bytes of static LDS", (size_t)a.sharedSizeBytes);
    return SABER_OK;
}
template <int PACK>
static int check_estep_lds_layout() {
    SABER_TRY(static_lds_is_zero(estep_kernel<MODE_SAMPLE, true, uint16_t, PACK>));
    SABER_TRY(static_lds_is_zero(estep_kernel<MODE_PROBS, true, uint16_t, PACK>));
    SABER_TRY(static_lds_is_zero(estep_kernel<MODE_LOGLIK, true, uint16_t, PACK>));
    SABER_TRY(static_lds_is_zero(estep_kernel<MODE_SAMPLE, true, int32_t, PACK>));
    SABER_TRY(static_lds_is_zero(estep_kernel<MODE_PROBS, true, int32_t, PACK>));
    SABER_TRY(static_lds_is_zero(estep_kernel<MODE_LOGLIK, true, int32_t, PACK>));
    if (PACK == PACK_16_14) SABER_TRY(static_lds_is_zero(estep_kernel<MODE_SAMPLE, true, uint16_t, PACK_16_14, true>));
    return SABER_OK;
}

// Wavefronts a CU holds of a sampling kernel with `block` threads per workgroup, given its LDS (handed out in 1,280-byte pieces) and
// the 32 wavefronts a CU can hold.  The choice of a workgroup's size (estep_auto_block(), tile_classes()) reckons with pieces of 512 bytes
// and 144 bytes on top instead, and just below its lines a CU then holds fewer wavefronts than it asks for: in chunks of 4 M
// tokens and more 20 at K = 6,613 to 6,640 and 16 at 13,229 to 13,316 (for 24), in smaller ones 21 at 1,569 to 1,724 (for 22), 20 at
// 3,461 to 3,612 (for 22) and 16 at 7,873 to 8,024 (for 20).  An iteration at T = 15 M: K = 5,700 1.26 ms, 6,630 1.39, 8,200 1.30; 11,500
// 1.43, 13,300 1.82, 15,000 1.60.
constexpr size_t kLdsPiece = 1280;
static int estep_waves_per_cu(const saber_ctx *c, int block, size_t piece = 512) {
    const size_t need = c->staged || c->overlay ? ((estep_lds_bytes(c, MODE_SAMPLE, block) + (piece == 512 ? 144 : 0) + piece - 1) / piece) * piece : 512;
    const int by_lds = (int)std::min<size_t>(64, (size_t)c->lds_per_cu / need), by_waves = 32 / (block / 64);
    return std::min(by_lds, by_waves) * (block / 64);
}

// Workgroups that n tiles of light words are dealt to, every so-manieth tile to each (the tiles are sorted by size: the shares are
// alike).  The Bhat rows of light words differ in a few topics, so a workgroup that works on several stages the base vector
// once and exchanges these topics: T = 15 M, K = 20,011, 80 KB per row and 90 tokens per tile, 2.03 ms per iteration with one
// tile per workgroup, 1.70, 1.67 and 1.72 with 4, 12 and 64; T = 36 M, K = 5,000 2.49, 2.40 with 4, 2.43 with 8 and 2.59 with
// 64; T = 100 M, K = 10,000 7.44, 7.28, 7.35 with 12 and 7.99 with 64.  What many per workgroup lose is the tail of
// the launch: every place on the chip gets 16 workgroups in turn or more, and 8 tiles are the most.  With
// rows of 4 and 8 KB (T = 10 M, K = 1,000; T = 20 M, K = 2,000) no number of tiles changes anything, so rows of 16 KB are the least.
// The log-likelihood pass has no registers for it, and gained nothing.
constexpr int64_t kWalkTiles = 8, kWalkRounds = 16;
constexpr size_t kWalkRow = 16 * 1024;
static int32_t walkers_for(const saber_ctx *c, int mode, int64_t n, int block) {
    if (!c->staged || !c->z16 || mode != MODE_SAMPLE || n <= 0 || estep_row_bytes(c) < kWalkRow) return (int32_t)n;
    const int64_t places = c->cus * estep_waves_per_cu(c, block, kLdsPiece) / (block / 64);   // (at least one workgroup fits: make_ctx() sees to it)
    const int64_t tiles = std::max<int64_t>(1, std::min(kWalkTiles, n / (kWalkRounds * places)));
    return (int32_t)((n + tiles - 1) / tiles);
}

// One E-step launch per tile class (tile_classes() below).  All stage the row in LDS when it fits.
// `theta`: the context whose rows of A are read, c itself but for the scored part of held-out documents.  What may be taken for
// granted of their entries is its knowledge: an observed part may be longer than any scored one.
template <int MODE>
static int launch_estep(saber_ctx *c, const saber_ctx *theta, const Chunk &ch, EStepParams &p0) {
    // (theta's documents are c's documents: same D, same chunks - the held-out contexts have one chunk each)
    set_rows(p0, theta, theta->chunks[(size_t)(&ch - c->chunks.data())]);
    for (const TileClass &cl : ch.classes) {
        for (int64_t i = 0, n; i < cl.count; i += n) {
            n = std::min(cl.count - i, most_blocks(cl.block));
            EStepParams p = p0;
            p.tiles = p0.tiles + cl.first + i;
            if (p0.out_ll) p.out_ll = p0.out_ll + cl.first + i;
            p.first_light = (int32_t)std::max<int64_t>(0, std::min(cl.n_dense - i, n));
            p.n_tiles = (int32_t)n;
            p.walkers = walkers_for(c, MODE, n - p.first_light, cl.block);
            const dim3 grid((unsigned)(p.first_light + p.walkers)), block((unsigned)cl.block);
            const size_t lds = estep_lds_bytes(c, MODE, cl.block);
            if (c->staged) {
                if (c->z16) launch_estep_packed<MODE, true, uint16_t>(c, theta->pack, grid, block, lds, p);
                else launch_estep_packed<MODE, true, int32_t>(c, theta->pack, grid, block, lds, p);
            } else {
                if (c->z16) launch_estep_packed<MODE, false, uint16_t>(c, theta->pack, grid, block, lds, p);
                else launch_estep_packed<MODE, false, int32_t>(c, theta->pack, grid, block, lds, p);
            }
            HIP_TRY(hipGetLastError());
        }
    }
    return SABER_OK;
}

// Threads of a sampling workgroup where the caller leaves them open.
//
// A staged row: the smallest workgroup with which LDS still lets a CU hold most of its 32 wavefronts.  A word's tile is dealt to
// the workgroup's wavefronts, and each pays its set-up (Philox for a few lanes, run boundaries, the chain of dependent loads)
// for its share: sampling pass at T = 20 M, 60,000 words, K from 1,200 to 9,500, always 32 wavefronts per CU: 1.17 ms with 64
// threads, 1.21 with 128, 1.30 with 256, 1.51 with 512, 1.93 with 1,024.  Fewer wavefronts cost: 28 of them 6 %, 24 11 %, 20
// 43 %, 16 45 %.  So a size is taken from 31, 28, 24, 20 wavefronts on, the more the larger the next size's loss.  In chunks
// below 4 M tokens the shares are small and the sizes further apart (T = 1.5 M, 15,000 words: 0.09, 0.11, 0.13, 0.17 and 0.27
// ms), and 22, 22, 20 and 16 wavefronts do.  T = 10 M, K = 1,000 0.68 -> 0.62 ms, T = 2.3 M, K = 777 0.15 -> 0.13, T = 20 M in
// four chunks, K = 2,000 2.3 -> 1.6, T = 100 M, K = 1,000 6.45 -> 6.29, all against 256 threads and launches by size of tile.
//
// With the caller's tile_tokens the tiles are not matched to the workgroup (below), and one wavefront may be left with the
// whole of a large one (T = 10 M, K = 73, tiles of 1,280 tokens: 0.53 ms with 64 threads, 0.44 with 128 or with tiles of
// 320): the size is then the one with the most wavefronts, ties to the smaller, and light words' tiles get launches by size.
//
// A row that is not staged is gathered through the caches: the more of a CU's wavefronts
// work on the same row the better, once it is too long for the 32 KB of a CU's L1 to hold several.  An iteration
// with 256, 512 and 1,024 threads at V = 50,000, T = 20 M: K = 300 2.03, 2.09 and 2.25 ms, K = 1,000 2.76, 2.69 and
// 2.81, K = 3,000 4.74, 4.00 and 3.47, K = 10,000 9.16, 7.00 and 6.01, K = 45,000 15.6, 12.9 and 10.6; at V = 100,000,
// T = 3 M, where most words have few tokens: K = 1,000 0.66, 0.77 and 0.98, K = 3,000 2.16, 2.07 and 2.26 in the
// first iterations and 1.41, 1.43 and 1.62 in later ones, K = 45,000 15.8, 13.8 and 12.7, and 6.98, 6.96 and 7.21.
//
// With marks for light words instead (Overlay) the base vector, which all of them share, fills the caches, and 256, 512 and
// 1,024 threads take 0.44, 0.45 and 0.48 ms at T = 1.5 M, K = 70,000, 0.91, 1.00 and 1.19 at T = 3 M, K = 45,000, but 8.7, 8.0 and
// 7.7 ms at T = 20 M, where the words with dense rows have most of the tokens (iterations 6 to 15).
constexpr int64_t kLargeChunk = 8ll << 20;
static int estep_auto_block(const saber_ctx *c, int64_t per_chunk) {
    if (c->overlay && per_chunk < kLargeChunk) return 256;
    if (!c->staged) return c->K <= 2048 ? 256 : 1024;
    if (c->tile_tokens_asked > 0) {
        int best = 256;
        for (int block : {512, 1024}) if (estep_waves_per_cu(c, block) > estep_waves_per_cu(c, best)) best = block;
        return best;
    }
    const bool small = per_chunk < (4ll << 20);
    const int least[4] = {small ? 22 : 31, small ? 22 : 28, small ? 20 : 24, small ? 16 : 20};
    for (int i = 0; i < 4; i++)
        if (estep_waves_per_cu(c, 64 << i) >= least[i]) return 64 << i;
    return 1024;
}

// Automatic tile size: a heavy word's Bhat row is staged once per tile, so larger tiles stage less; but a tile is
// the work of one workgroup (its wavefronts take it 64 tokens at a time), and the pass waits for its largest ones.
// A 32,768th of the chunk per wavefront of the workgroup, at most an 8192th and at most 32,768 tokens.  With 256 threads the
// sampling pass took 0.36 / 0.10 ms with tiles of 8,192 / 128
// tokens at T = 1 M, K = 300, 1.15 / 0.89 ms with 8,192 / 1,024 at 10 M, K = 1,000, 2.43 / 2.34 ms with 14,000 /
// 4,096 at 36 M, K = 5,000, and 9.14 / 9.06 ms with 32,768 / 8,192 at 100 M, K = 10,000 (512 threads); with 64 threads 0.53 /
// 0.43 ms with 1,280 / 320 at 10 M, K = 73, and 7.31 / 6.30 / 6.29 with 12,160 / 3,008 / 1,472 at 100 M, K = 1,000.
// A small tile has to be worth its row, though: not below K / 16 tokens, 64 to 256 (T = 300,000, K = 10,000: 0.072 ms with
// 64, 0.058 with 256).
static int32_t auto_tile_tokens(const saber_ctx *c, int64_t per_chunk) {
    // (a vocabulary of more than 2^19 words makes a tile or more per word as it is: larger tiles keep a chunk's within
    // the 2^20 of saber_loglik_static)
    const bool many_words = c->V > (1 << 19);
    // (likewise where documents are longer than the share of a chunk: it then has as many tokens as the longest more)
    const int64_t longest = (((per_chunk + c->max_doc_len) >> 19) + 64) & ~63ll;
    const int64_t least = many_words ? 8192 : std::max<int64_t>(longest, std::min<int64_t>(256, std::max<int64_t>(64, (c->K / 16) & ~63)));
    const int waves = c->staged ? std::min(4, c->opt.block_threads / 64) : 4;
    const int64_t share = many_words ? (per_chunk / 2560) & ~255ll : (per_chunk * waves / 32768) & ~63ll;
    return (int32_t)std::min<int64_t>(32768, std::max<int64_t>(least, share));
}

// Cuts a chunk's tiles - n_dense of words with dense rows, then those of light words, each group sorted by decreasing size -
// into classes.  Dense rows: tiles with at least stage_min_tokens tokens get block_threads threads, smaller ones
// light_block_threads.  Light words get light_block_threads as well, and one launch takes all tiles where the two are equal, as
// they are by default.  With the caller's tile_tokens, unless the caller fixed a workgroup size: one wavefront per 64 tokens
// (a full batch), between the smallest workgroup with which LDS still lets a CU hold 24 of its 32 wavefronts and block_threads
// (K = 1,000, T = 10 M, 90,000 light words of 29 tokens on average: 0.89 ms with 256 threads for all of them, 0.77 ms so).  Up
// to two rounds of the chip's 8,192 wavefronts that makes no difference (T = 2 M, K = 777: 0.17 ms both), and the light
// words' tiles then go with the dense rows' launch.
static void tile_classes(const saber_ctx *c, Chunk &ch, const Tile *tiles, int64_t n_dense) {
    int64_t at = 0;
    auto add = [&](int64_t to, int block) {
        if (to <= at) return;
        const int64_t dense = std::max<int64_t>(0, std::min(to, n_dense) - at);
        TileClass *last = ch.classes.empty() ? nullptr : &ch.classes.back();
        if (last && last->block == block) { last->count += to - at; last->n_dense += dense; }
        else ch.classes.push_back(TileClass{at, to - at, dense, block});
        at = to;
    };
    auto until = [&](int64_t end, int64_t least) {   // first tile from `at` to `end` with fewer than `least` tokens
        return (int64_t)(std::lower_bound(tiles + at, tiles + end, least, [](const Tile &t, int64_t n) { return t.count >= n; }) - tiles);
    };
    if (c->opt.stage_min_tokens > 1) add(until(n_dense, c->opt.stage_min_tokens), c->opt.block_threads);
    else add(n_dense, c->opt.block_threads);
    add(n_dense, c->opt.light_block_threads);
    int lo = c->opt.light_block_threads, hi = c->opt.light_block_threads;
    if (c->auto_light_block && c->tile_tokens_asked > 0 && ch.ntiles - n_dense > 16384) { lo = 64; while (lo < hi && estep_waves_per_cu(c, lo) < 24) lo *= 2; }
    for (int block = hi; block > lo; block /= 2) {
        const int64_t to = until(ch.ntiles, 64 * (block / 128) + 1);   // tiles that half the workgroup would not serve in one batch each
        if (to - at >= 128 || (block == hi && !ch.classes.empty() && ch.classes.back().block == hi)) add(to, block);   // (a launch of its own pays from half a workgroup per CU on)
    }
    add(ch.ntiles, lo);
}

// Every row of A is fetched once per word of its document, by the frequent words' tiles about a hundred times in a pass, and
// in a large chunk from beyond L2 (14 % hits at T = 100 M).  So the tiles of frequent words are cut at the ends of
// kDocRanges ranges of documents and launched range by range, each XCD (workgroups go to them round robin) at a range of
// its own at a time, whose rows its 4 MB L2 holds in part.  Sampling pass, iterations 11..20: T = 100 M, K = 10,000 7.92 ->
// 7.21 ms, K = 1,000 7.46 -> 6.48; T = 246 M in three chunks, K = 5,000, short documents 15.6 -> 14.4, 240 M of long ones,
// K = 10,000 26.5 -> 23.8; T = 36 M, K = 5,000 2.27 -> 2.14.  8 or 32 ranges gain half to all of that.  A word is cut if
// its pieces have 64 tokens on average (32 to 512 differ by 1 to 3 %).  Words that are not cut come first: at the end of the
// launch their larger tiles cost 3 to 5 %.  Where it stops:
//   * chunks whose rows of A the eight L2s hold together (32 MB, taken from the rows' capacities), and chunks below 8 M
//     tokens, where the pieces are small and 16 times the tiles weigh more than the traffic they save.  Change of the pass by
//     the cut, per cent, iterations 1..5 / 18..37: T = 4.5 M, rows of 13 to 18 MB (K = 300 to 1,000) +2..+4 / +1..+5, of
//     28 MB (short documents) +3..+5 / +1..+4; 8 M tokens, 33 MB -4..-1 / +1..+3, 37 MB -2..+3 / -2..+1, 50 MB (short
//     documents) +2..+5 / -3..0; 12 M, 18 MB +1 / +1, 55 MB -3..+1 / -6..0; 24 M, 68 to 110 MB -8..-2 / -7..-3.  The
//     number of topics alone does not tell: K = 300, 1,000 and 2,500 differ by 1 to 3 where the rows are alike;
//   * above K = 16,384 the rows are too long (K = 20,011, T = 15 M: first iterations 4.75 -> 5.02 ms, later ones 1.82 -> 1.79), and
//     rows that are not staged (K = 45,000, T = 20 M) lose the sharing of a row between tiles: 8.9 -> 9.9 ms;
//   * classes by size (stage_min_tokens) need the tiles in order of size;
//   * a chunk's tiles have to stay within the 2^20 of saber_loglik_static whatever the words' sizes are: one per word or piece
//     of a word, and one more per tile_tokens tokens.
constexpr int kXcds = 8, kDocRanges = 16;
constexpr int64_t kRangeTokens = 8ll << 20, kRangeRowUnits = (32ll << 20) / 128, kRangePiece = 64;

static bool may_cut_by_range(const saber_ctx *c, const Chunk &ch) {
    return c->staged && c->K <= 16384 && c->opt.stage_min_tokens <= 1 && ch.ntok >= kRangeTokens && ch.row_units >= kRangeRowUnits &&
           (int64_t)c->V + (int64_t)kDocRanges * c->V_dense + std::max<int64_t>(1 << 16, ch.ntok / c->opt.tile_tokens) <= 1 << 20;
}

// tiles[0, n) sorted by decreasing size -> the order of the launch: tile i
// is the next one of XCD i mod 8, which takes the ranges congruent to its number one after the other; uncut tiles first.
static void order_tiles_by_range(Tile *tiles, int64_t n) {
    std::vector<Tile> list[kXcds], out;
    out.reserve((size_t)n);
    for (int64_t i = 0; i < n; i++) (tiles[i].range ? list[(tiles[i].range - 1) % kXcds] : out).push_back(tiles[i]);
    for (auto &l : list) std::stable_sort(l.begin(), l.end(), [](const Tile &a, const Tile &b) { return a.range < b.range; });
    size_t at[kXcds] = {};
    while ((int64_t)out.size() < n) {
        int x = (int)(out.size() % kXcds);
        if (at[x] == list[x].size()) for (x = 0; at[x] == list[x].size(); x++) {}   // its ranges are done: what another has left
        out.push_back(list[x][at[x]++]);
    }
    std::copy(out.begin(), out.end(), tiles);
}

// Tiles of dense-row words first, then those of light words; inside each group heavy tiles first, so the tail of a launch is made
// of small ones (Sec. 3.4), and equal ones in the order they have.  Returns the number of the first kind.  (Counted into place: by
// comparisons 30,000 tiles took 0.9 ms.)
constexpr int32_t kTileBins = 1 << 16;
static int64_t sort_tiles(std::vector<Tile> &tiles, size_t first, const std::vector<int32_t> &word_row) {
    const size_t n = tiles.size() - first;
    int32_t most = 0;
    int64_t n_dense = 0;
    for (size_t i = first; i < tiles.size(); i++) { most = std::max(most, tiles[i].count); n_dense += word_row[(size_t)tiles[i].word] >= 0; }
    if (most >= kTileBins) {   // (larger tiles than the default's are the caller's)
        std::stable_sort(tiles.begin() + (ptrdiff_t)first, tiles.end(), [&](const Tile &a, const Tile &b) {
            const bool la = word_row[(size_t)a.word] < 0, lb = word_row[(size_t)b.word] < 0;
            return la != lb ? lb : a.count > b.count;
        });
        return n_dense;
    }
    auto bin = [&](const Tile &t) { return (size_t)(most - t.count) + (word_row[(size_t)t.word] < 0 ? (size_t)most + 1 : 0); };
    std::vector<size_t> at(2 * (size_t)most + 3, 0);
    for (size_t i = first; i < tiles.size(); i++) at[bin(tiles[i]) + 1]++;
    for (size_t b = 1; b < at.size(); b++) at[b] += at[b - 1];
    std::vector<Tile> sorted(n);
    for (size_t i = first; i < tiles.size(); i++) sorted[at[bin(tiles[i])]++] = tiles[i];
    std::copy(sorted.begin(), sorted.end(), tiles.begin() + (ptrdiff_t)first);
    return n_dense;
}

// Segmented count of up to two groupings of the assignments: documents over z (CountByDZ -> rows of A) and light words
// over z_wm (CountByVZ -> sparse rows of B).  Two launches: short segments with one wavefront each, long ones
// with 256 threads.
struct SegLists { SegGroup g; const int32_t *short_list; int64_t n_short; const int32_t *long_list; int64_t n_long; };
static int launch_segmented_count(saber_ctx *c, const SegLists &a, const SegLists &b) {
    for (int pass = 0; pass < 2; pass++) {
        const int64_t na = pass == 0 ? a.n_short : a.n_long, nb = pass == 0 ? b.n_short : b.n_long;
        const int block = pass == 0 ? 64 : 256;
        if (na + nb == 0) continue;
        SegGroup ga = a.g, gb = b.g;
        ga.list = pass == 0 ? a.short_list : a.long_list; gb.list = pass == 0 ? b.short_list : b.long_list;
        // LDS: bitmap + rank prefix (2 * nwords) + the row under construction; a short segment's row has at
        // most long_doc_tokens entries, so its workgroup asks for no more than that
        const int budget = std::max(0, (int)((63 * 1024 - 8 * (int64_t)c->nwords) / 4));
        const int want = pass == 0 ? std::min(c->opt.long_doc_tokens, c->K) : c->opt.dz_lds_entries;
        const int entries = std::min(want, budget);
        const size_t lds = ((size_t)2 * c->nwords + (size_t)entries) * sizeof(uint32_t);
        if (lds > 63 * 1024) {   // K > 2^17: the two bitmap arrays alone pass 64 KB; gfx950 has 160 KB per workgroup
            const void *fn = c->z16 ? (const void *)count_dz_kernel<uint16_t> : (const void *)count_dz_kernel<int32_t>;
            HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        }
        for (int64_t i = 0, n; i < na + nb; i += n) {   // segments [i, i + n) of the two lists in a row
            n = std::min(na + nb - i, most_blocks(block));
            const int64_t left = std::max<int64_t>(0, std::min(i + n, na) - i);   // of the first list
            SegGroup pa = ga, pb = gb;
            if (left) pa.list += i; else pb.list += i - na;
            const dim3 grid((unsigned)n), blk((unsigned)block);
            if (c->z16)
                hipLaunchKernelGGL((count_dz_kernel<uint16_t>), grid, blk, lds, c->stream, pa, left, pb, c->count_bits, c->nwords, entries);
            else
                hipLaunchKernelGGL((count_dz_kernel<int32_t>), grid, blk, lds, c->stream, pa, left, pb, c->count_bits, c->nwords, entries);
            HIP_TRY(hipGetLastError());
        }
    }
    return SABER_OK;
}
static SegLists light_segments(const saber_ctx *c) {
    return SegLists{{nullptr, c->light_tok_ptr, c->z_wm, 0, c->wrec, c->lw_ent}, c->light_short, c->n_light_short, c->light_long, c->n_light_long};
}
// the rows of B of a model's light words; held-out documents borrow theirs and count none
static SegLists own_light_segments(const saber_ctx *c) { return c->parent ? SegLists{} : light_segments(c); }

// Ablation: A rebuilt by sorting the (document, topic) pairs of all tokens
static int launch_sort_rebuild(saber_ctx *c) {
    if (c->T == 0 || c->D == 0) return SABER_OK;
    const dim3 grid((unsigned)((c->D + 3) / 4)), block(256);
    if (c->z16)
        hipLaunchKernelGGL((sort_keys_kernel<uint16_t>), grid, block, 0, c->stream, c->doc_ptr, (const uint16_t *)c->z, c->D,
                           c->topic_bits, c->sort_keys);
    else
        hipLaunchKernelGGL((sort_keys_kernel<int32_t>), grid, block, 0, c->stream, c->doc_ptr, (const int32_t *)c->z, c->D,
                           c->topic_bits, c->sort_keys);
    HIP_TRY(hipGetLastError());
    size_t bytes = c->sort_tmp_bytes;
    HIP_TRY(rocprim::radix_sort_keys(c->sort_tmp, bytes, c->sort_keys, c->sort_keys_out, (size_t)c->T, 0u, c->sort_end_bit,
                                     c->stream));
    hipLaunchKernelGGL(sort_mark_kernel, grid, block, 0, c->stream, c->doc_ptr, c->sort_keys_out, c->D, c->count_bits,
                       c->docrec, c->cd_ent, c->sort_rank);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(sort_count_kernel, grid, block, 0, c->stream, c->doc_ptr, c->sort_rank, c->D, c->docrec, c->cd_ent);
    HIP_TRY(hipGetLastError());
    return SABER_OK;
}

// CountByDZ of all documents, and CountByVZ of the light words
static int launch_counts(saber_ctx *c) {
    if (c->opt.ablation & 2) {
        SABER_TRY(launch_sort_rebuild(c));
        return launch_segmented_count(c, SegLists{}, own_light_segments(c));
    }
    return launch_segmented_count(c, SegLists{{nullptr, c->doc_ptr, c->z, 0, c->docrec, c->cd_ent}, c->short_docs, c->n_short,
                                              c->long_docs, c->n_long}, own_light_segments(c));
}

// CountByDZ for the documents of one chunk whose assignments sit in a buffer
static int launch_count_dz_chunk(saber_ctx *c, const Chunk &ch, int slot) {
    const ZView zv = z_view(c, ch, slot);
    return launch_segmented_count(c, SegLists{{nullptr, c->doc_ptr, zv.z, zv.first, c->docrec, c->cd_ent}, c->short_docs + ch.short0,
                                              ch.nshort, c->long_docs + ch.long0, ch.nlong}, SegLists{});
}

// ---- host streaming ----
static int sync_all(saber_ctx *c) {
    HIP_TRY(hipStreamSynchronize(c->stream));
    if (c->n_slots) { HIP_TRY(hipStreamSynchronize(c->s_in)); HIP_TRY(hipStreamSynchronize(c->s_docs)); }
    return SABER_OK;
}
// Takes the next buffer (round robin) for chunk `ch`: once the kernels of the buffer's previous user have run, the chunk's tok_t is
// copied in, and with `docs` tok_doc derived from it.  stream_wait() makes the compute stream wait for that.
static int stream_load(saber_ctx *c, const Chunk &ch, bool docs, int *slot) {
    const int s = c->next_slot;
    c->next_slot = (c->next_slot + 1) % c->n_slots;
    if (ch.ntok > c->slot_tokens) return fail(SABER_ESTATE, "chunk of %lld tokens exceeds the streaming buffers", (long long)ch.ntok);
    // (a call that broke off between here and stream_release() has left work on any of the three streams that no event tells of)
    if (c->slot_open[s]) SABER_TRY(sync_all(c));
    else if (c->slot_used[s]) HIP_TRY(hipStreamWaitEvent(c->s_in, c->ev_done[s], 0));
    c->slot_open[s] = true;
    *slot = s;
    if (ch.ntok == 0) return SABER_OK;
    HIP_TRY(hipMemcpyAsync(c->slot_tok_t[s], c->h_tok_t + ch.t0, (size_t)ch.ntok * sizeof(uint32_t), hipMemcpyHostToDevice, c->s_in));
    HIP_TRY(hipEventRecord(docs ? c->ev_copied[s] : c->ev_loaded[s], c->s_in));
    if (!docs) return SABER_OK;
    // on a stream of its own: the look-ups of this kernel wait for memory most of the time and run beside the sampling of the
    // chunk before (1.7 ms per 123 M tokens of short documents when it ran in line with it), and the next chunk's copy, which
    // has nothing to wait for, goes on (T = 20 M in four chunks, K = 2,000, the link the slower one: 1.63 -> 1.54 ms
    // per iteration)
    HIP_TRY(hipStreamWaitEvent(c->s_docs, c->ev_copied[s], 0));
    hipLaunchKernelGGL(expand_tok_doc_kernel, dim3(grid_for(ch.ntok, 256)), dim3(256), 0, c->s_docs, c->slot_tok_t[s],
                       ch.ntok, ch.t0, c->doc_blocks, c->ne_doc, c->slot_tok_doc[s]);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipEventRecord(c->ev_loaded[s], c->s_docs));
    return SABER_OK;
}
static int stream_wait(saber_ctx *c, const Chunk &ch, int s) {
    if (ch.ntok) HIP_TRY(hipStreamWaitEvent(c->stream, c->ev_loaded[s], 0));
    return SABER_OK;
}
static int stream_acquire(saber_ctx *c, const Chunk &ch, int *slot, bool docs = true) {
    SABER_TRY(stream_load(c, ch, docs, slot));
    return stream_wait(c, ch, *slot);
}
// After the chunk's kernels have been queued: the buffer may be overwritten once they have run.
static int stream_release(saber_ctx *c, int s) {
    HIP_TRY(hipEventRecord(c->ev_done[s], c->stream));
    c->slot_used[s] = true;
    c->slot_open[s] = false;
    return SABER_OK;
}

// Preprocess + BuildTree for the light words (sparse rows of B); needs the base vector, i.e. runs after launch_phi
static LightParams light_params(const saber_ctx *c) {
    return LightParams{c->light_words, c->wrec, c->lw_ent, c->lw_phi, c->denom, c->phi + (size_t)c->V_dense * (size_t)c->Kpad,
                       c->l3_64 + (size_t)c->V * (size_t)c->n3, c->l3, c->l3_64, c->sumphi, c->n3, c->n3pad, c->V_light, c->n_light_wide, c->count_bits, c->beta};
}
// Light words per wavefront: four where rows are short enough that their chain of loads counts (up to 128 blocks of topics) and the
// chip stays full of wavefronts.  Kernel with one, two and four, late iterations: T = 10 M, K = 1,000, 98,600 words (dense rows with
// them) 35, 29 and 28 us; T = 2.3 M, K = 777, 29,500 words 12.5, 11.3 and 11.2; T = 36 M, K = 5,000, 140,000 words 76, 70 and 69; T =
// 100 M, K = 10,000 119, 118 and 121; T = 15 M, K = 20,011 104, 106 and 123; T = 1.5 M, K = 70,000, 4,000 words 38, 69 and 126; T = 100 K
// 5.6 all.
//   A word has a step of 64 non-zeros after the other, and those of four words come one after the other: the first iterations, and
// words that the caller keeps light, have thousands.  So words of more than kWideWord tokens (four steps, as a wavefront of four
// words has then too) have a wavefront each, before the others.  Phi group with one word, with four, and so, iterations 2 to 4 / late: T =
// 6 M, K = 8,000, 60,000 words 51 / 40, 109 / 54 and 51 / 39 us; T = 2 M, K = 4,000, 30,000 words 24 / 18, 59 / 25 and 23 / 17; T = 10 M,
// K = 1,000 40 / 36, 32 / 29 and 34 / 30; T = 3 M, K = 5,000, all of 20,000 words light 83 / 51, 260 / 129 and 81 / 52.  (Lines at 64 and at
// 512 tokens are 0 to 2 us slower late, and in the first iterations.)  The words of many tokens have the first numbers: a list cost 0.4 to
// 1.3 us, marks 1 to 4.
constexpr int64_t kWideWord = 256;
static int words_per_wave(const saber_ctx *c) { return c->n3 <= 128 && c->V_light - c->n_light_wide >= 16384 ? 4 : 1; }
static unsigned light_waves(const saber_ctx *c) {
    const int per_wave = words_per_wave(c);
    return (unsigned)(c->n_light_wide + (c->V_light - c->n_light_wide + per_wave - 1) / per_wave);
}
static int launch_light_words(saber_ctx *c) {
    if (c->V_light == 0) return SABER_OK;
    hipLaunchKernelGGL((words_per_wave(c) == 4 ? light_tree_kernel<4> : light_tree_kernel<1>), dim3(light_waves(c)), dim3(64), light_lds_bytes(c->n3),
                       c->stream, light_params(c));
    HIP_TRY(hipGetLastError());
    return SABER_OK;
}

// dense-branch tokens (slots, or null), nnz(A), sum_d K_d L_d, sum_d K_d U_d and the non-zeros of the sparse rows of B
// (what the next E-step will read) into five device counters
static StatsParams stats_params(const saber_ctx *c, const unsigned long long *slots, unsigned long long *out) {
    return StatsParams{slots, slots ? kDenseSlots : 0, c->docrec, c->doc_ptr, c->doc_words, c->D, c->wrec, c->V_light, out};
}
static int stats_blocks(const saber_ctx *c, int block) { return grid_for(std::max<int64_t>(c->D, c->V_light), block, 256); }
static int launch_stats(saber_ctx *c, const unsigned long long *slots, unsigned long long *out) {
    hipLaunchKernelGGL(stats_kernel, dim3(stats_blocks(c, 256)), dim3(256), 0, c->stream, stats_params(c, slots, out));
    HIP_TRY(hipGetLastError());
    return SABER_OK;
}

// Topics of one workgroup's LDS histogram: at most 36,864 (144 of the CU's 160 KB); more topics are shared out evenly over
// the grid's y.
constexpr int kHistTopics = 36 * 1024;
static int hist_range(const saber_ctx *c) {
    const int ranges = (c->K + kHistTopics - 1) / kHistTopics;
    return ((c->K + ranges - 1) / ranges + 63) / 64 * 64;
}
static int allow_lds(const void *kernel, size_t lds) {   // more than the default 64 KB has to be asked for
    if (lds > 64 * 1024) HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    return SABER_OK;
}

// B and the accumulators of the topic totals, all zero.  An M-step finds them so, as the one before left them; a new
// context, or one in which a call broke off in between, clears them first.
static int launch_clear_accumulators(saber_ctx *c, bool totals) {
    const size_t vk = ((size_t)c->V_dense + 1) * (size_t)c->Kpad;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for((int64_t)vk, 256, 8192)), dim3(256), 0, c->stream, (uint32_t *)c->cwk, 0u, vk);
    HIP_TRY(hipGetLastError());
    if (totals) {
        hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(2 * (int64_t)c->K + 1, 256)), dim3(256), 0, c->stream, (uint32_t *)c->ck_acc, 0u, (size_t)c->K * 2 + 1);
        HIP_TRY(hipGetLastError());
    }
    c->acc_used = false;
    return SABER_OK;
}

// The first n_items slabs of the dense rows' segments into B (rows all zero on entry), and with `totals` the histogram of
// all assignments into the accumulators of the topic totals.
static int launch_count_slabs(saber_ctx *c, int64_t n_items, bool totals) {
    if (c->acc_used) SABER_TRY(launch_clear_accumulators(c, true));
    // Counting in LDS, by ranges of topics, replaces one global atomic per token where K is too large for one histogram:
    // totals 0.74 -> 0.04 ms and rows 0.39 -> 0.04 ms at T = 15 M, K = 20,011, 0.13 -> 0.04 and 0.24 -> 0.03 ms at
    // T = 1.5 M, K = 70,000.
    const int range = hist_range(c);
    // every workgroup ends with up to K atomics into the K totals: no more than about 500 shares of z (128 where these
    // have fewer than 65,536 assignments: T = 10 M, K = 1,000 takes 17 us with 153 of them, 21 with 490), none with
    // fewer than 16 assignments per topic (but 16,384 at least, and 131,072 are enough at any K: a late iteration at T = 1.5 M,
    // K = 70,000 0.41 ms with 262,144, 0.39 with 131,072, 0.40 with 65,536 and 0.41 with fewer, at T = 15 M, K = 20,011 1.66, 1.65, 1.66
    // and 1.66) or more than 2^20, keep those from dominating
    const int64_t least = std::max<int64_t>(16384, std::min<int64_t>(16 * (int64_t)c->K, 131072));
    const int64_t share = std::max<int64_t>(c->T / 512, std::min<int64_t>(c->T / 128, 65536));
    const int64_t per_block = std::min<int64_t>(1 << 20, std::max<int64_t>(least, ((share + 4095) / 4096) * 4096));
    const int64_t n_tot = totals ? (c->T + per_block - 1) / per_block : 0;
    if (n_tot + n_items == 0) return SABER_OK;
    const size_t lds = (size_t)std::min(range, c->K) * 4;
    // a histogram of all assignments: their order does not matter, and with host streaming the word-major copy is
    // the one that is resident
    const void *zsrc = c->n_slots ? c->z_wm : c->z;
    SABER_TRY(allow_lds(c->z16 ? (const void *)count_slabs_kernel<uint16_t> : (const void *)count_slabs_kernel<int32_t>, lds));
    c->acc_used = true;
    for (int64_t i = 0, n; i < n_tot + n_items; i += n) {
        n = std::min(n_tot + n_items - i, most_blocks(1024));
        const int tot = i == 0 ? (int)n_tot : 0;   // (far fewer than a launch takes: all in the first one)
        const VzItem *items = c->vz_items + (i == 0 ? 0 : i - n_tot);
        const dim3 grid((unsigned)n, (unsigned)((c->K + range - 1) / range));
        if (c->z16)
            hipLaunchKernelGGL((count_slabs_kernel<uint16_t>), grid, dim3(1024), lds, c->stream, (const uint16_t *)zsrc, c->T, per_block,
                               tot, c->ck_acc, items, (const uint16_t *)c->z_wm, c->cwk, c->K, c->Kpad, range);
        else
            hipLaunchKernelGGL((count_slabs_kernel<int32_t>), grid, dim3(1024), lds, c->stream, (const int32_t *)zsrc, c->T, per_block,
                               tot, c->ck_acc, items, (const int32_t *)c->z_wm, c->cwk, c->K, c->Kpad, range);
        HIP_TRY(hipGetLastError());
    }
    return SABER_OK;
}

// LDS of one workgroup of the alias-table build: K + 1 prefix sums (binary64) and K item numbers
static size_t alias_lds_bytes(int K) { return ((size_t)K + 1) * sizeof(double) + (size_t)K * sizeof(uint32_t); }

// Threads of a phi_tree_kernel workgroup: a column for each of its four per step
static int phi_block_threads(const saber_ctx *c) { return c->Kpad <= 1024 ? 256 : c->Kpad <= 2048 ? 512 : 1024; }

// Which contexts' M-steps take two launches instead of seven or eight: those with light words, resident, and small.  An iteration
// that way and the other: T = 100 K, K = 100 30 and 38 us; 1 M, K = 21 75 and 103; 1.9 M, K = 44 98 and 120; 2.3 M, K = 777 162 and
// 181; 10 M, K = 1,000 649 and 671; 10.8 M in 207,000 documents, K = 73 519 and 544.  Not with more topics than 4,096, where the last
// workgroup of the totals takes longer than the launches saved (T = 725 K, K = 3,000 84 and 92 us, 5,612 99 and 96, 14,000 174 and
// 156), nor with more segments (T = 36 M, 535,000 documents and light words: 2,604 and 2,577): wavefronts that share a workgroup
// hold their places until the last is done.
constexpr int kJoinedTopics = 4096;
constexpr int64_t kJoinedSegments = 384 * 1024, kJoinedTokens = 16ll << 20;
// Assignments of one share of the totals, or of one slab, in a joined M-step (its workgroups have 256 threads, and every share
// ends with K atomics, a fence and a ticket): T = 2.3 M, K = 777 182, 177, 169, 161 us per iteration with 4, 8, 17, 48 thousand;
// T = 10 M, K = 1,000 649 with T / 48, 653 with T / 32, 686 with T / 20.
static int64_t joined_share(const saber_ctx *c) { return std::max<int64_t>(std::max<int64_t>(16384, std::min(16 * c->K, 65536)), (c->T / 48 + 4095) & ~4095ll); }

// A row of several ranges of topics has a workgroup for each, and a second launch for the running sums, where one workgroup per row
// would leave CUs without any.  Phi group without and with, late iterations at T = 1.5 M: K = 8,257 61 rows 28.0 and 25.9 us, 255 25.3 and
// 24.0; K = 20,011 37.9 and 31.5, 34.9 and 31.2; K = 60,000 71 and 45, 66 and 49.  The gain does not end at that line: 301 and 501 rows
// 27.8 and 24.5, 28.4 and 26.4 at K = 8,257, 75 and 51, 75 and 61 at K = 60,000; more rows, and larger corpora, were not measured.
static int launch_phi(saber_ctx *c) {
    hipLaunchKernelGGL(denominators_kernel, dim3(grid_for(c->Kpad, 256)), dim3(256), 0, c->stream, c->ck_acc, c->ck, c->denom, c->K,
                       c->Kpad, c->vbeta);
    HIP_TRY(hipGetLastError());
    // kPhiSteps steps of four columns per thread at a time: up to 8,192 topics (32 KB of LDS; a CU holds two workgroups of
    // 1,024 threads, by its 32 wavefronts)
    const dim3 block((unsigned)phi_block_threads(c));
    const int range = std::min(c->Kpad, kPhiSteps * 4 * (int)block.x);
    const size_t hist = (size_t)range * sizeof(uint32_t);
    const int64_t rows = (int64_t)c->V_dense + 1;
    const int parts = (c->Kpad + range - 1) / range;
    const bool by_parts = parts > 1 && rows <= c->cus;
    for (int64_t r = 0, n; r < rows; r += n) {
        n = std::min(rows - r, most_blocks((int)block.x));
        const dim3 grid((unsigned)n, by_parts ? (unsigned)parts : 1u);
        const size_t at = (size_t)r * (size_t)c->Kpad;
        auto launch = [&](auto kernel, auto *z_wm) {
            hipLaunchKernelGGL(kernel, grid, block, hist, c->stream, c->phi_rows + r, z_wm, c->cwk + at, c->denom, c->phi + at, c->l3, c->l3_64, c->sumphi,
                               c->Kpad, c->n3, c->n3pad, c->beta, range);
        };
        if (c->z16) launch(by_parts ? phi_tree_kernel<uint16_t, true> : phi_tree_kernel<uint16_t, false>, (const uint16_t *)c->z_wm);
        else launch(by_parts ? phi_tree_kernel<int32_t, true> : phi_tree_kernel<int32_t, false>, (const int32_t *)c->z_wm);
        HIP_TRY(hipGetLastError());
    }
    if (by_parts) {
        hipLaunchKernelGGL(phi_sums_kernel, dim3((unsigned)rows), dim3(256), ((size_t)c->n3 + (size_t)(c->n3 + 15) / 16) * sizeof(double), c->stream,
                           c->phi_rows, c->l3, c->l3_64, c->sumphi, c->n3, c->n3pad);
        HIP_TRY(hipGetLastError());
    }
    c->acc_used = false;
    if (c->alias_table && c->V_dense > 0) {   // measurement variant: an alias table per word on top of the tree level
        const size_t lds = alias_lds_bytes(c->K);
        if (lds > 64 * 1024)
            HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(alias_sweep_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(alias_sweep_kernel, dim3((unsigned)c->V_dense), dim3(kAliasThreads), lds, c->stream, c->phi, c->K, c->Kpad, c->alias_table);
        HIP_TRY(hipGetLastError());
    }
    return SABER_OK;
}

// The M-step of a small corpus: all counts in one launch, all that follows from them in another (see MCounts).
static int launch_joined_mstep(saber_ctx *c, const unsigned long long *slots, unsigned long long *stats_out, hipEvent_t counted) {
    if (c->acc_used) SABER_TRY(launch_clear_accumulators(c, true));
    MCounts p{};
    p.docs = SegGroup{c->long_docs, c->doc_ptr, c->z, 0, c->docrec, c->cd_ent}; p.short_docs = c->short_docs;
    p.words = SegGroup{c->light_long, c->light_tok_ptr, c->z_wm, 0, c->wrec, c->lw_ent}; p.short_words = c->light_short;
    p.n_long_docs = (int)c->n_long; p.n_short_docs = (int)c->n_short;
    p.n_long_words = (int)c->n_light_long; p.n_short_words = (int)c->n_light_short;
    p.T = c->T; p.per_block = joined_share(c); p.n_tot = (int)((c->T + p.per_block - 1) / p.per_block); p.n_items = (int)c->n_vz_long;
    p.acc = c->ck_acc; p.ck = c->ck; p.ticket = (unsigned *)(c->ck_acc + c->K);
    p.items = c->vz_items; p.cwk = c->cwk;
    p.count_bits = c->count_bits; p.nwords = c->nwords; p.lds_entries = std::min(c->opt.dz_lds_entries, c->K); p.wave_entries = std::min(c->opt.long_doc_tokens, c->K);
    p.vbeta = c->vbeta; p.beta = c->beta; p.denom = c->denom; p.phi = c->phi; p.l3 = c->l3; p.sumphi = c->sumphi; p.l3_64 = c->l3_64;
    p.K = c->K; p.Kpad = c->Kpad; p.n3 = c->n3; p.n3pad = c->n3pad; p.range = std::min(c->Kpad, kPhiSteps * 4 * 256);
    p.base_row = c->V_dense; p.base_word = c->V;
    const int64_t n_short = (int64_t)p.n_short_docs + p.n_short_words;
    const int64_t grid = (int64_t)p.n_tot + p.n_items + p.n_long_docs + p.n_long_words + (n_short + 3) / 4;
    const size_t lds = 4 * std::max({(size_t)c->Kpad, (size_t)2 * c->nwords + (size_t)p.lds_entries, 4 * ((size_t)2 * c->nwords + (size_t)p.wave_entries)});
    SABER_TRY(allow_lds((const void *)mstep_counts_kernel, lds));
    c->acc_used = true;
    hipLaunchKernelGGL(mstep_counts_kernel, dim3((unsigned)grid), dim3(256), lds, c->stream, p);
    HIP_TRY(hipGetLastError());
    if (counted) HIP_TRY(hipEventRecord(counted, c->stream));
    const int block = phi_block_threads(c), nw = block / 64, range = std::min(c->Kpad, kPhiSteps * 4 * block);
    const LightParams lp = light_params(c);
    const StatsParams st = stats_params(c, slots, stats_out);
    const int n_stats = stats_blocks(c, block);
    const unsigned grid2 = (unsigned)(n_stats + c->V_dense) + (light_waves(c) + nw - 1) / nw;
    const size_t lds2 = std::max((size_t)range * 4, (size_t)nw * light_lds_bytes(c->n3));
    hipLaunchKernelGGL((words_per_wave(c) == 4 ? mstep_rows_kernel<4> : mstep_rows_kernel<1>), dim3(grid2), dim3((unsigned)block), lds2, c->stream, c->phi_rows, c->V_dense,
                       (const uint16_t *)c->z_wm, c->cwk, c->phi, c->Kpad, range, st, n_stats, lp);
    HIP_TRY(hipGetLastError());
    c->acc_used = false;
    return SABER_OK;
}

// Word-major copy of z (after init / set_z; an E-step writes it itself).
static int launch_fill_zwm_chunk(saber_ctx *c, const Chunk &ch, int slot) {
    if (ch.ntiles == 0) return SABER_OK;
    const uint32_t *tok_t = slot < 0 ? c->tok_t + ch.t0 : c->slot_tok_t[slot];
    const ZView zv = z_view(c, ch, slot);
    if (c->z16)
        hipLaunchKernelGGL((fill_zwm_kernel<uint16_t>), dim3((unsigned)ch.ntiles), dim3(256), 0, c->stream,
                           c->tiles + ch.tile0, tok_t, (const uint16_t *)zv.z, ch.t0 - zv.first, (uint16_t *)c->z_wm);
    else
        hipLaunchKernelGGL((fill_zwm_kernel<int32_t>), dim3((unsigned)ch.ntiles), dim3(256), 0, c->stream,
                           c->tiles + ch.tile0, tok_t, (const int32_t *)zv.z, ch.t0 - zv.first, (int32_t *)c->z_wm);
    HIP_TRY(hipGetLastError());
    return SABER_OK;
}
static int launch_fill_zwm(saber_ctx *c) {
    for (const Chunk &ch : c->chunks) SABER_TRY(launch_fill_zwm_chunk(c, ch, -1));
    return SABER_OK;
}

// Ablation: the E-step over the tokens in document order, then the word-major copy from z
static int launch_estep_docmajor(saber_ctx *c, unsigned long long *n_dense) {
    if (c->T == 0 || c->D == 0) return SABER_OK;
    DocMajorParams p{};
    p.doc_ptr = c->doc_ptr; p.word_ids = c->word_ids_d; p.word_row = c->word_row_d;
    p.docrec = c->docrec; p.cd_ent = c->cd_ent;
    p.phi = c->phi; p.l3 = c->l3; p.sumphi = c->sumphi; p.l3_64 = c->l3_64;
    p.z = c->z; p.n_dense = n_dense; p.D = c->D;
    p.K = c->K; p.Kpad = c->Kpad; p.n3 = c->n3; p.n3pad = c->n3pad;
    p.count_bits = c->count_bits; p.alpha = c->alpha;
    p.seed_lo = (uint32_t)c->seed; p.seed_hi = (uint32_t)(c->seed >> 32); p.iter = c->iter;
    const dim3 grid((unsigned)((c->D + 3) / 4)), block(256);
    if (c->z16) hipLaunchKernelGGL((estep_docmajor_kernel<uint16_t>), grid, block, 0, c->stream, p);
    else hipLaunchKernelGGL((estep_docmajor_kernel<int32_t>), grid, block, 0, c->stream, p);
    HIP_TRY(hipGetLastError());
    return launch_fill_zwm(c);
}

// iteration 0: the Philox draw of Alg. 1's initialisation for the canonical tokens [t0, t1), stored from z[z_rel] on
static int launch_init_z(saber_ctx *c, void *z, int64_t z_rel, int64_t t0, int64_t t1) {
    if (t1 <= t0) return SABER_OK;
    if (c->z16)
        hipLaunchKernelGGL((init_z_kernel<uint16_t>), dim3(grid_for(t1 - t0, 256, 8192)), dim3(256), 0, c->stream,
                           (uint16_t *)z, z_rel, t0, t1, (uint32_t)c->K, (uint32_t)c->seed, (uint32_t)(c->seed >> 32));
    else
        hipLaunchKernelGGL((init_z_kernel<int32_t>), dim3(grid_for(t1 - t0, 256, 8192)), dim3(256), 0, c->stream,
                           (int32_t *)z, z_rel, t0, t1, (uint32_t)c->K, (uint32_t)c->seed, (uint32_t)(c->seed >> 32));
    HIP_TRY(hipGetLastError());
    return SABER_OK;
}

// The M-step after the assignments changed outside an E-step: all four rebuilds of Alg. 1.
// With host streaming the assignments are not on the device: they come chunk by chunk from user_z, or when that
// is null from the Philox draw of iteration 0.
static int full_mstep(saber_ctx *c, const int32_t *user_z = nullptr) {
    if (c->n_slots) {   // chunk by chunk: rows of A and the word-major copy
        std::vector<uint16_t> stage;
        for (const Chunk &ch : c->chunks) {
            int s;
            SABER_TRY(stream_acquire(c, ch, &s, false));
            if (user_z && ch.ntok) {
                HIP_TRY(hipStreamSynchronize(c->stream));   // the buffer's earlier kernels are done: plain copy
                const void *src = user_z + ch.t0;
                if (c->z16) {
                    stage.resize((size_t)ch.ntok);
                    for (int64_t i = 0; i < ch.ntok; i++) stage[(size_t)i] = (uint16_t)user_z[ch.t0 + i];
                    src = stage.data();
                }
                HIP_TRY(hipMemcpy(c->slot_z[s], src, (size_t)ch.ntok * (c->z16 ? 2 : 4), hipMemcpyHostToDevice));
            } else {
                SABER_TRY(launch_init_z(c, c->slot_z[s], 0, ch.t0, ch.t0 + ch.ntok));
            }
            SABER_TRY(launch_count_dz_chunk(c, ch, s));
            SABER_TRY(launch_fill_zwm_chunk(c, ch, s));
            SABER_TRY(stream_release(c, s));
        }
        SABER_TRY(launch_segmented_count(c, SegLists{}, own_light_segments(c)));
    } else {
        if (!c->parent) SABER_TRY(launch_fill_zwm(c));
        if (!c->joined) SABER_TRY(launch_counts(c));
    }
    if (c->parent) {   // held-out documents: A only, the model stays frozen
        HIP_TRY(hipStreamSynchronize(c->stream));
        return SABER_OK;
    }
    // with the workload numbers of the E-step that will read the new A: nnz(A), sum_d K_d * L_d, ...
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, c->stream, (uint32_t *)c->counters, 0u, (size_t)kCtr * 2);
    HIP_TRY(hipGetLastError());
    if (c->joined) {
        SABER_TRY(launch_joined_mstep(c, nullptr, c->counters, nullptr));
    } else {
        SABER_TRY(launch_count_slabs(c, c->n_vz_long, true));
        SABER_TRY(launch_phi(c));
        SABER_TRY(launch_light_words(c));
        SABER_TRY(launch_stats(c, nullptr, c->counters));
    }
    SABER_TRY(sync_all(c));
    unsigned long long h[kCtr];
    HIP_TRY(hipMemcpy(h, c->counters, sizeof(h), hipMemcpyDeviceToHost));
    c->stats.nnz_cd = (int64_t)h[1]; c->stats.next_row_entries = (int64_t)h[2]; c->stats.next_row_fetch = (int64_t)h[3];
    c->stats.next_light_entries = (int64_t)h[4];
    return SABER_OK;
}

// ------------------------------------------------------------------------------------------------
// saber_init
// ------------------------------------------------------------------------------------------------
// What lay_out() makes on the host and upload() takes to the device.
struct Layout {
    std::vector<int32_t> row_word, light_words, light_short, light_long, short_docs, long_docs;
    std::vector<int64_t> light_tok_ptr = std::vector<int64_t>(1, 0);
    std::vector<uint2> wrec, docrec;
    std::vector<VzItem> vz_items;
    std::vector<PhiRow> phi_rows;
    // the word-major token arrays: ordinary host memory on the way to the device, or with host streaming the pinned array that
    // stays (tok_doc is then derived on the device)
    std::vector<int32_t> v_tok_doc; std::vector<uint32_t> v_tok_t;
    int32_t *tok_doc = nullptr; uint32_t *tok_t = nullptr;
    std::vector<Tile> tiles;
    std::vector<uint32_t> doc_words;
};

// (For a context on a trained model no call of the runtime is made: another thread may do it.)
static int lay_out(saber_ctx *c, const int64_t *doc_ptr, const int32_t *word_ids, Layout &lay) {
    const int64_t D = c->D, T = c->T; const int32_t V = c->V, K = c->K;
    auto &h_row_word = lay.row_word, &h_light_words = lay.light_words, &h_light_short = lay.light_short, &h_light_long = lay.light_long;
    auto &h_light_tok_ptr = lay.light_tok_ptr;
    auto &h_wrec = lay.wrec;
    auto &h_vz_items = lay.vz_items; auto &h_phi_rows = lay.phi_rows;
    int32_t *&h_tok_doc = lay.tok_doc; uint32_t *&h_tok_t = lay.tok_t;
    auto &v_tok_doc = lay.v_tok_doc; auto &v_tok_t = lay.v_tok_t;
    auto &h_tiles = lay.tiles;
    auto &h_rec = lay.docrec; auto &h_short = lay.short_docs, &h_long = lay.long_docs;
    auto &h_doc_words = lay.doc_words;
    // ---- chunks: contiguous document ranges of about equal token count (Sec. 3.1.2) ----
    // A chunk also ends before its rows of A (128-byte aligned slots of capacity min(L_d, K)) would pass 4 GB: the
    // sampling kernel addresses them by 32-bit byte offsets.  That only happens with far fewer chunks than the default.
    const int nch = std::max(1, c->opt.n_chunks);
    const int64_t unit_limit = (int64_t)0xfff00000ll / 128;
    c->chunks.clear();
    {
        int64_t d = 0;
        for (int i = 0; i < nch || d < D; i++) {
            Chunk ch; ch.d0 = d; ch.t0 = doc_ptr[d];
            const int64_t target = i < nch - 1 ? (T * (int64_t)(i + 1)) / nch : T;
            int64_t units = 0;
            while (d < D && doc_ptr[d + 1] <= target) {
                const int64_t u = (std::min<int64_t>(doc_ptr[d + 1] - doc_ptr[d], K) + 31) / 32;
                if (units + u > unit_limit) break;
                units += u; d++;
            }
            ch.d1 = d; ch.ntok = doc_ptr[d] - ch.t0; ch.row_units = units;
            if (ch.ntok >= (1ll << 31)) return fail(SABER_ERANGE, "saber_init: a document chunk holds %lld tokens (limit 2^31)", (long long)ch.ntok);
            if (ch.d1 > ch.d0) c->chunks.push_back(ch);
        }
    }
    // ---- words: dense rows of B for the frequent ones, sparse rows for the rest ----
    // A word with n tokens has at most n non-zero counts; below light_word_tokens tokens its sparse row
    // (8 bytes per non-zero, rebuilt by a segmented count like a row of A) is cheaper than 12*K bytes of dense B / Bhat
    // traffic per iteration.  Needs a Bhat row in LDS (16-bit assignments, then), or marks in LDS where it cannot hold a row (Overlay).
    const bool light_ok = (c->staged ? c->z16 : c->overlay) && c->opt.light_word_tokens > 0;
    const saber_ctx *par = c->parent;   // then the model's word classes are taken over
    c->joined = light_ok && c->z16 && !par && c->n_slots == 0 && c->opt.ablation == 0 && K <= kJoinedTopics && D + V <= kJoinedSegments && T <= kJoinedTokens;
    // (as many counts as a packed entry of a sparse row has bits for)
    c->opt.light_word_tokens = std::min(c->opt.light_word_tokens, 1 << std::min(16u, c->count_bits));
    std::vector<int64_t> n_v;
    if (par) {
        c->h_word_row = par->h_word_row;
        c->V_dense = par->V_dense; c->V_light = par->V_light;
    } else {
        n_v.assign((size_t)V, 0);
        for (int64_t t = 0; t < T; t++) n_v[(size_t)word_ids[t]]++;
        c->h_word_row.assign((size_t)V, 0);
        // Light rows lie in the order of the vocabulary, as an export writes them (by number it went over the caller's pages twice: 6.3 ->
        // 10.1 ms for B of 60,000 words at K = 1,000); those of words with many tokens have the first numbers: see words_per_wave().
        int64_t lunits = 0;
        std::vector<std::pair<int32_t, uint32_t>> wide, narrow;   // word, row start
        for (int32_t v = 0; v < V; v++) {
            if (light_ok && n_v[(size_t)v] < c->opt.light_word_tokens) {
                if (lunits > 0xffffffffll) return fail(SABER_ERANGE, "sparse rows of B exceed 2^32 * 128 bytes");
                (n_v[(size_t)v] > kWideWord ? wide : narrow).emplace_back(v, (uint32_t)lunits);
                lunits += (std::min<int64_t>(n_v[(size_t)v], K) + 31) / 32;
            } else {
                c->h_word_row[(size_t)v] = (int32_t)h_row_word.size();
                h_row_word.push_back(v);
            }
        }
        c->n_light_wide = (int32_t)wide.size();
        for (const auto *list : {&wide, &narrow}) for (const auto &[v, unit] : *list) {
            const int32_t li = (int32_t)h_light_words.size();
            c->h_word_row[(size_t)v] = -li - 1;
            h_light_words.push_back(v);
            h_light_tok_ptr.push_back(h_light_tok_ptr.back() + n_v[(size_t)v]);
            h_wrec.push_back(make_uint2(unit, 0u));
            (n_v[(size_t)v] > c->opt.long_doc_tokens ? h_light_long : h_light_short).push_back(li);
        }
        c->V_dense = (int32_t)h_row_word.size(); c->V_light = (int32_t)h_light_words.size();
        h_row_word.push_back(V);   // the all-zero row: its Bhat is the base vector, its tree level the base running sums
        c->T_light = h_light_tok_ptr.back(); c->lw_cap = lunits * 32;
        c->n_light_short = (int64_t)h_light_short.size(); c->n_light_long = (int64_t)h_light_long.size();
    }
    // ---- resident or streamed?  stream_workers = 0 keeps everything on the device when it fits and falls back to
    // host streaming with three buffers when it does not ----
    if (!par && c->opt.stream_workers == 0 && c->opt.ablation == 0 && T > 0) {
        const size_t zs = c->z16 ? 2 : 4;
        size_t row_units = 0, slot_tokens = 0, tiles_bound = (size_t)(T / std::max(1, c->opt.tile_tokens));
        for (int64_t d = 0; d < D; d++) row_units += (size_t)((std::min<int64_t>(doc_ptr[d + 1] - doc_ptr[d], K) + 31) / 32);
        for (const Chunk &ch : c->chunks) {
            slot_tokens = std::max(slot_tokens, (size_t)ch.ntok);
            tiles_bound += (size_t)std::min<int64_t>(V, ch.ntok);
            if (may_cut_by_range(c, ch)) tiles_bound += (size_t)std::min<int64_t>((int64_t)kDocRanges * c->V_dense, ch.ntok / kRangePiece);
        }
        const size_t common = row_units * 128 + (size_t)D * 32 + tiles_bound * sizeof(Tile) +
                              ((size_t)c->V_dense + 1) * (size_t)c->Kpad * 8 +
                              ((size_t)V + 1) * ((size_t)c->n3pad * 4 + (size_t)c->n3 * 8 + 4) + (size_t)c->lw_cap * 8 +
                              (size_t)T * zs + ((size_t)32 << 20);
        const size_t resident = common + (size_t)T * (8 + zs);
        const size_t streamed = common + 3 * slot_tokens * (8 + zs) + (size_t)T / 4 + (size_t)D * 4;
        size_t limit = (size_t)std::max(0, c->opt.device_mem_limit_mb) << 20;
        if (limit == 0) {
            size_t free_b = 0, total_b = 0;
            HIP_TRY(hipMemGetInfo(&free_b, &total_b));
            limit = free_b;
        }
        if (resident > limit - limit / 16) {
            if (streamed > limit - limit / 16)
                return fail(SABER_ENOMEM, "saber_init: the corpus needs about %.1f GB of device memory (%.1f GB with the token "
                            "lists streamed from the host) and %.1f GB are available; more chunks shrink the streaming buffers",
                            resident / 1e9, streamed / 1e9, limit / 1e9);
            c->n_slots = 3;
        }
    }
    c->stats.stream_workers = c->n_slots;
    c->joined = c->joined && c->n_slots == 0 && c->V_light > 0 && T > 0;

    // ---- word-major token arrays and tiles per chunk (host counting sort; layout only) ----
    // position of every word's segment in the word-major order (light words first, then dense rows) and the
    // slabs CountByVZ cuts the dense rows' segments into
    // (on a trained model nobody reads the word-major assignments: they lie as the tokens do.  The sampling kernel folds in as it
    // trains, and writes them all the same: 1.1 MB in a row per iteration of 550,000 tokens, 0.2 us, are not worth a test per batch)
    std::vector<int64_t> wm_ptr, wm_seen;   // wm_seen: tokens placed so far (chunk by chunk)
    // phi_tree_kernel counts a row itself up to 32 tokens per thread of its workgroup; longer rows are cut into slabs for
    // count_slabs_kernel (phi group of T = 2.3 M, K = 777, 256 threads: 43 us with 8,192 tokens, 49 with 32,768; of T = 100 M,
    // K = 10,000, 1,024 threads: 343 us counting none, 323 with 8,192, 303 with 32,768, 298 with 131,072)
    const int64_t own_tokens = 32 * phi_block_threads(c);
    if (!par) {
        wm_ptr.assign((size_t)V, 0); wm_seen.assign((size_t)V, 0);
        for (int32_t li = 0; li < c->V_light; li++) wm_ptr[(size_t)h_light_words[(size_t)li]] = h_light_tok_ptr[(size_t)li];
        int64_t pos = c->T_light;
        const int64_t slab = c->joined ? joined_share(c) : 131072;
        for (int32_t r = 0; r < c->V_dense; r++) {
            const int32_t v = h_row_word[(size_t)r];
            wm_ptr[(size_t)v] = pos;
            h_phi_rows.push_back(PhiRow{v, n_v[(size_t)v] <= own_tokens ? (int32_t)n_v[(size_t)v] : -1, pos});
            for (int64_t s = 0; s < n_v[(size_t)v]; s += slab)
                h_vz_items.push_back(VzItem{r, (int32_t)std::min<int64_t>(slab, n_v[(size_t)v] - s), pos + s});
            pos += n_v[(size_t)v];
        }
        h_phi_rows.push_back(PhiRow{V, 0, 0});
        c->n_vz_long = std::stable_partition(h_vz_items.begin(), h_vz_items.end(), [&](const VzItem &it) {
                           return h_phi_rows[(size_t)it.row].count < 0; }) - h_vz_items.begin();
        c->n_vz_items = (int64_t)h_vz_items.size();
    }
    if (c->n_slots) {
        const size_t n = (size_t)std::max<int64_t>(T, 1);
        HIP_TRY(hipHostMalloc((void **)&c->h_tok_t, n * sizeof(uint32_t), hipHostMallocDefault));
        h_tok_doc = nullptr; h_tok_t = c->h_tok_t;   // tok_doc is derived on the device
    } else {
        v_tok_doc.resize((size_t)std::max<int64_t>(T, 1)); v_tok_t.resize((size_t)std::max<int64_t>(T, 1));
        h_tok_doc = v_tok_doc.data(); h_tok_t = v_tok_t.data();
    }
    std::vector<int64_t> wcount((size_t)V + 1);
    const int tile_tokens = c->opt.tile_tokens;
    for (Chunk &ch : c->chunks) {
        std::fill(wcount.begin(), wcount.end(), 0);
        for (int64_t t = ch.t0; t < ch.t0 + ch.ntok; t++) wcount[(size_t)word_ids[t] + 1]++;
        for (int32_t v = 0; v < V; v++) wcount[(size_t)v + 1] += wcount[(size_t)v];
        const size_t first_tile = h_tiles.size();
        for (int64_t d = ch.d0; d < ch.d1; d++)
            for (int64_t t = doc_ptr[d]; t < doc_ptr[d + 1]; t++) {
                const int64_t pos = ch.t0 + wcount[(size_t)word_ids[t]]++;
                if (h_tok_doc) h_tok_doc[(size_t)pos] = (int32_t)d;
                h_tok_t[(size_t)pos] = (uint32_t)(t - ch.t0);
            }
        // ranges of documents: see order_tiles_by_range()
        const bool ranges = may_cut_by_range(c, ch);
        const int n_ranges = ranges ? kDocRanges : 1;
        std::vector<uint32_t> range_end((size_t)n_ranges, 0u);   // tokens of the chunk up to the end of each range
        int64_t rd = ch.d0;
        for (int r = 0; r < n_ranges; r++) {
            const int64_t target = ch.t0 + ch.ntok * (r + 1) / n_ranges;
            while (rd < ch.d1 && (r == n_ranges - 1 || doc_ptr[rd + 1] <= target)) rd++;
            range_end[(size_t)r] = (uint32_t)(doc_ptr[rd] - ch.t0);
        }
        for (int32_t v = 0; v < V; v++) {
            const int64_t b = v ? wcount[(size_t)v - 1] : 0, e = wcount[(size_t)v];   // (the starts have moved to the ends)
            const int32_t row = c->h_word_row[(size_t)v];
            if (e > b) { ch.words_present++; if (row < 0) c->stats.light_words_present++; }
            const bool split = n_ranges > 1 && row >= 0 && e - b >= n_ranges * kRangePiece;
            int64_t s = b;
            for (int r = 0; r < (split ? n_ranges : 1); r++) {
                const uint32_t *seg = h_tok_t + ch.t0;   // (ascending inside a word's segment)
                const int64_t end = split ? std::lower_bound(seg + s, seg + e, range_end[(size_t)r]) - seg : e;
                while (s < end) {
                    const int32_t cnt = (int32_t)std::min<int64_t>(tile_tokens, end - s);
                    h_tiles.push_back(Tile{v, (int32_t)s, cnt, row >= 0 ? row : -row - 1, par ? ch.t0 + s : wm_ptr[(size_t)v] + wm_seen[(size_t)v], split ? r + 1 : 0});
                    if (!par) wm_seen[(size_t)v] += cnt;
                    s += cnt;
                }
            }
        }
        // tiles of dense-row words first, then those of light words; inside each group heavy tiles first so the
        // tail of a launch is made of small ones (Sec. 3.4)
        const int64_t n_dense = sort_tiles(h_tiles, first_tile, c->h_word_row);
        if (n_ranges > 1) order_tiles_by_range(h_tiles.data() + first_tile, n_dense);
        ch.tile0 = (int64_t)first_tile; ch.ntiles = (int64_t)(h_tiles.size() - first_tile);
        tile_classes(c, ch, h_tiles.data() + first_tile, n_dense);
        c->max_chunk_tiles = std::max(c->max_chunk_tiles, ch.ntiles);
    }
    c->total_tiles = (int64_t)h_tiles.size();
    // ---- rows of A: fixed, 128-byte aligned slots of capacity min(L_d, K) (Sec. 3.4 aligns rows likewise) ----
    h_rec.resize((size_t)std::max<int64_t>(D, 1));
    if (!par) {   // distinct words per document (layout statistic for the bandwidth model)
        h_doc_words.resize((size_t)std::max<int64_t>(D, 1));
        std::vector<int32_t> last_doc((size_t)V, -1);
        for (int64_t d = 0; d < D; d++) {
            uint32_t u = 0;
            for (int64_t t = doc_ptr[d]; t < doc_ptr[d + 1]; t++) {   // (no branch: repeats are irregular)
                int32_t &last = last_doc[(size_t)word_ids[t]];
                u += last != (int32_t)d;
                last = (int32_t)d;
            }
            h_doc_words[(size_t)d] = u;
        }
    }
    c->doc_len.resize((size_t)D);
    int64_t units = 0;
    for (int64_t d = 0; d < D; d++) {
        const int64_t len = doc_ptr[d + 1] - doc_ptr[d];
        c->doc_len[(size_t)d] = len;
        if (units > 0xffffffffll) return fail(SABER_ERANGE, "rows of A exceed 2^32 * 128 bytes");
        h_rec[(size_t)d] = make_uint2((uint32_t)units, 0u);
        units += (std::min<int64_t>(len, K) + 31) / 32;
        (len > c->opt.long_doc_tokens ? h_long : h_short).push_back((int32_t)d);
    }
    c->cd_cap = units * 32;
    c->n_short = (int64_t)h_short.size(); c->n_long = (int64_t)h_long.size();
    for (Chunk &ch : c->chunks) {   // both lists ascend by document: a chunk's documents are a contiguous part of each
        ch.row_unit0 = (int64_t)h_rec[(size_t)ch.d0].x;
        ch.short0 = std::lower_bound(h_short.begin(), h_short.end(), (int32_t)ch.d0) - h_short.begin();
        ch.nshort = (std::lower_bound(h_short.begin(), h_short.end(), (int32_t)std::min<int64_t>(ch.d1, 0x7fffffff)) - h_short.begin()) - ch.short0;
        ch.long0 = std::lower_bound(h_long.begin(), h_long.end(), (int32_t)ch.d0) - h_long.begin();
        ch.nlong = (std::lower_bound(h_long.begin(), h_long.end(), (int32_t)std::min<int64_t>(ch.d1, 0x7fffffff)) - h_long.begin()) - ch.long0;
        c->slot_tokens = std::max(c->slot_tokens, ch.ntok);
    }

    return SABER_OK;
}

static int upload(saber_ctx *c, const int64_t *doc_ptr, const int32_t *word_ids, const Layout &lay) {
    const int64_t D = c->D, T = c->T; const int32_t V = c->V, K = c->K;
    const saber_ctx *par = c->parent;
    const auto &h_row_word = lay.row_word, &h_light_words = lay.light_words, &h_light_short = lay.light_short, &h_light_long = lay.light_long;
    const auto &h_light_tok_ptr = lay.light_tok_ptr;
    const auto &h_wrec = lay.wrec;
    const auto &h_vz_items = lay.vz_items; const auto &h_phi_rows = lay.phi_rows;
    const int32_t *h_tok_doc = lay.tok_doc; const uint32_t *h_tok_t = lay.tok_t;
    const auto &h_tiles = lay.tiles;
    const auto &h_rec = lay.docrec; const auto &h_short = lay.short_docs, &h_long = lay.long_docs;
    const auto &h_doc_words = lay.doc_words;
    if (c->hooks.have_stream) { c->stream = c->hooks.stream; c->own_stream = false; }
    else { HIP_TRY(hipStreamCreate(&c->stream)); c->own_stream = true; }
    if (c->opt.profile) {
        for (auto &e : c->ev) HIP_TRY(hipEventCreate(&e));
        c->have_events = true;
    }
    // ---- device memory (what a context without assignments of its own never reads stays out) ----
    const bool state = !c->no_state;
    const size_t vk = ((size_t)c->V_dense + 1) * (size_t)c->Kpad;
    if (c->n_slots) {
        HIP_TRY(hipStreamCreateWithFlags(&c->s_in, hipStreamNonBlocking));
        HIP_TRY(hipStreamCreateWithFlags(&c->s_docs, hipStreamNonBlocking));
        for (int s = 0; s < c->n_slots; s++) {
            SABER_TRY(dev_alloc(c->hooks, &c->slot_tok_doc[s], (size_t)c->slot_tokens)); SABER_TRY(dev_alloc(c->hooks, &c->slot_tok_t[s], (size_t)c->slot_tokens));
            if (c->z16) SABER_TRY(dev_alloc(c->hooks, (uint16_t **)&c->slot_z[s], (size_t)c->slot_tokens));
            else SABER_TRY(dev_alloc(c->hooks, (int32_t **)&c->slot_z[s], (size_t)c->slot_tokens));
            HIP_TRY(hipEventCreateWithFlags(&c->ev_copied[s], hipEventDisableTiming));
            HIP_TRY(hipEventCreateWithFlags(&c->ev_loaded[s], hipEventDisableTiming));
            HIP_TRY(hipEventCreateWithFlags(&c->ev_done[s], hipEventDisableTiming));
        }
        std::vector<uint4> blocks((size_t)((T + 63) / 64) + 1, make_uint4(0u, 0u, 0u, 0u));
        std::vector<int32_t> ne;
        for (int64_t d = 0; d < D; d++) {
            const int64_t t = doc_ptr[d], end = doc_ptr[d + 1];
            if (end <= t) continue;
            const uint32_t r = (uint32_t)ne.size();
            ne.push_back((int32_t)d);
            const int j = (int)(t & 63);
            if (j) { uint4 &q = blocks[(size_t)(t >> 6)]; if (j < 32) q.y |= 1u << j; else q.z |= 1u << (j - 32); }
            for (int64_t b = (t + 63) >> 6; b <= (end - 1) >> 6; b++) blocks[(size_t)b].x = r;   // blocks that begin inside d
        }
        SABER_TRY(dev_alloc(c->hooks, &c->doc_blocks, blocks.size()));
        HIP_TRY(hipMemcpy(c->doc_blocks, blocks.data(), sizeof(uint4) * blocks.size(), hipMemcpyHostToDevice));
        if ((int64_t)ne.size() != D) {   // some document is empty: ordinals are not document numbers
            SABER_TRY(dev_alloc(c->hooks, &c->ne_doc, ne.size()));
            if (!ne.empty()) HIP_TRY(hipMemcpy(c->ne_doc, ne.data(), sizeof(int32_t) * ne.size(), hipMemcpyHostToDevice));
        }
    } else {
        if (state) {
            if (c->z16) SABER_TRY(dev_alloc(c->hooks, (uint16_t **)&c->z, (size_t)T)); else SABER_TRY(dev_alloc(c->hooks, (int32_t **)&c->z, (size_t)T));
        }
        SABER_TRY(dev_alloc(c->hooks, &c->tok_doc, (size_t)T)); SABER_TRY(dev_alloc(c->hooks, &c->tok_t, (size_t)T));
    }
    SABER_TRY(dev_alloc(c->hooks, &c->tiles, h_tiles.size())); SABER_TRY(dev_alloc(c->hooks, &c->doc_ptr, (size_t)D + 1));
    if (state) {
        SABER_TRY(dev_alloc(c->hooks, &c->docrec, (size_t)D)); SABER_TRY(dev_alloc(c->hooks, &c->cd_ent, (size_t)c->cd_cap));
        SABER_TRY(dev_alloc(c->hooks, &c->short_docs, h_short.size())); SABER_TRY(dev_alloc(c->hooks, &c->long_docs, h_long.size()));
    }
    if (par) {
        // borrowed from the model: everything the sampler reads about words
        c->phi = par->phi; c->l3 = par->l3; c->l3_64 = par->l3_64; c->sumphi = par->sumphi;
        c->wrec = par->wrec; c->lw_ent = par->lw_ent; c->lw_phi = par->lw_phi;
    } else {
    SABER_TRY(dev_alloc(c->hooks, &c->cwk, vk)); SABER_TRY(dev_alloc(c->hooks, &c->ck, (size_t)K)); SABER_TRY(dev_alloc(c->hooks, &c->ck_acc, (size_t)K + 1)); SABER_TRY(dev_alloc(c->hooks, &c->denom, (size_t)c->Kpad));
    SABER_TRY(dev_alloc(c->hooks, &c->phi, vk)); SABER_TRY(dev_alloc(c->hooks, &c->l3_64, ((size_t)V + 1) * (size_t)c->n3));
    SABER_TRY(dev_alloc(c->hooks, &c->row_word, h_row_word.size())); SABER_TRY(dev_alloc(c->hooks, &c->light_words, h_light_words.size()));
    SABER_TRY(dev_alloc(c->hooks, &c->light_short, h_light_short.size())); SABER_TRY(dev_alloc(c->hooks, &c->light_long, h_light_long.size()));
    SABER_TRY(dev_alloc(c->hooks, &c->light_tok_ptr, h_light_tok_ptr.size())); SABER_TRY(dev_alloc(c->hooks, &c->wrec, h_wrec.size()));
    SABER_TRY(dev_alloc(c->hooks, &c->lw_ent, (size_t)c->lw_cap)); SABER_TRY(dev_alloc(c->hooks, &c->lw_phi, (size_t)c->lw_cap));
    }
    if (state) {
        if (c->z16) SABER_TRY(dev_alloc(c->hooks, (uint16_t **)&c->z_wm, (size_t)T)); else SABER_TRY(dev_alloc(c->hooks, (int32_t **)&c->z_wm, (size_t)T));
    }
    if (!par) {
    SABER_TRY(dev_alloc(c->hooks, &c->vz_items, h_vz_items.size())); SABER_TRY(dev_alloc(c->hooks, &c->phi_rows, h_phi_rows.size()));
    HIP_TRY(hipMemcpy(c->phi_rows, h_phi_rows.data(), sizeof(PhiRow) * h_phi_rows.size(), hipMemcpyHostToDevice));
    if (!h_vz_items.empty())
        HIP_TRY(hipMemcpy(c->vz_items, h_vz_items.data(), sizeof(VzItem) * h_vz_items.size(), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(c->row_word, h_row_word.data(), sizeof(int32_t) * h_row_word.size(), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(c->light_tok_ptr, h_light_tok_ptr.data(), sizeof(int64_t) * h_light_tok_ptr.size(), hipMemcpyHostToDevice));
    }
    if (c->V_light && !par) {
        HIP_TRY(hipMemcpy(c->light_words, h_light_words.data(), sizeof(int32_t) * h_light_words.size(), hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(c->wrec, h_wrec.data(), sizeof(uint2) * h_wrec.size(), hipMemcpyHostToDevice));
        if (!h_light_short.empty()) HIP_TRY(hipMemcpy(c->light_short, h_light_short.data(), sizeof(int32_t) * h_light_short.size(), hipMemcpyHostToDevice));
        if (!h_light_long.empty()) HIP_TRY(hipMemcpy(c->light_long, h_light_long.data(), sizeof(int32_t) * h_light_long.size(), hipMemcpyHostToDevice));
    }
    if (!par) SABER_TRY(dev_alloc(c->hooks, &c->doc_words, (size_t)D));
    if (c->opt.ablation & 1) {
        SABER_TRY(dev_alloc(c->hooks, &c->word_ids_d, (size_t)T)); SABER_TRY(dev_alloc(c->hooks, &c->word_row_d, (size_t)V));
        if (T) HIP_TRY(hipMemcpy(c->word_ids_d, word_ids, sizeof(int32_t) * (size_t)T, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(c->word_row_d, c->h_word_row.data(), sizeof(int32_t) * (size_t)V, hipMemcpyHostToDevice));
    }
    if (c->opt.ablation & 4)
        SABER_TRY(dev_alloc(c->hooks, &c->alias_table, (size_t)std::max(c->V_dense, 1) * (size_t)K));
    if (c->opt.ablation & 2) {
        unsigned dbits = 1; while (dbits < 32 && (1ll << dbits) < std::max<int64_t>(D, 1)) dbits++;
        c->sort_end_bit = c->topic_bits + dbits;
        SABER_TRY(dev_alloc(c->hooks, &c->sort_keys, (size_t)T)); SABER_TRY(dev_alloc(c->hooks, &c->sort_keys_out, (size_t)T));
        SABER_TRY(dev_alloc(c->hooks, &c->sort_rank, (size_t)T));
        size_t bytes = 0;
        HIP_TRY(rocprim::radix_sort_keys(nullptr, bytes, c->sort_keys, c->sort_keys_out, (size_t)std::max<int64_t>(T, 1), 0u,
                                         c->sort_end_bit, c->stream));
        c->sort_tmp_bytes = std::max<size_t>(bytes, 1);
        SABER_TRY(hook_alloc(c->hooks, &c->sort_tmp, c->sort_tmp_bytes));
    }
    if (!par) { SABER_TRY(dev_alloc(c->hooks, &c->l3, ((size_t)V + 1) * (size_t)c->n3pad)); SABER_TRY(dev_alloc(c->hooks, &c->sumphi, (size_t)V + 1)); }
    if (!par) SABER_TRY(dev_alloc(c->hooks, &c->counters, (size_t)kMaxTimedIters * kCtr));
    if (state) SABER_TRY(dev_alloc(c->hooks, &c->dense_slots, (size_t)(par ? 1 : kMaxTimedIters) * kDenseSlots));
    if (!par || !state) SABER_TRY(dev_alloc(c->hooks, &c->ll_partial, (size_t)std::max<int64_t>(c->max_chunk_tiles, 1) + kLlTail));
    if (T && !c->n_slots) {
        HIP_TRY(hipMemcpy(c->tok_doc, h_tok_doc, sizeof(int32_t) * (size_t)T, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(c->tok_t, h_tok_t, sizeof(uint32_t) * (size_t)T, hipMemcpyHostToDevice));
    }
    if (!h_tiles.empty()) HIP_TRY(hipMemcpy(c->tiles, h_tiles.data(), sizeof(Tile) * h_tiles.size(), hipMemcpyHostToDevice));
    if (D && state) HIP_TRY(hipMemcpy(c->docrec, h_rec.data(), sizeof(uint2) * (size_t)D, hipMemcpyHostToDevice));
    if (D && !par) HIP_TRY(hipMemcpy(c->doc_words, h_doc_words.data(), sizeof(uint32_t) * (size_t)D, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(c->doc_ptr, doc_ptr, sizeof(int64_t) * ((size_t)D + 1), hipMemcpyHostToDevice));
    if (state && !h_short.empty()) HIP_TRY(hipMemcpy(c->short_docs, h_short.data(), sizeof(int32_t) * h_short.size(), hipMemcpyHostToDevice));
    if (state && !h_long.empty()) HIP_TRY(hipMemcpy(c->long_docs, h_long.data(), sizeof(int32_t) * h_long.size(), hipMemcpyHostToDevice));
    c->stats.tokens = T; c->stats.tiles = c->total_tiles; c->stats.chunks = (int64_t)c->chunks.size();
    if (c->no_state) { HIP_TRY(hipStreamSynchronize(c->stream)); return SABER_OK; }

    // ---- iteration 0: Philox assignment, then the M-step ----
    if (!c->n_slots) SABER_TRY(launch_init_z(c, c->z, 0, 0, T));   // with host streaming: chunk by chunk, in full_mstep
    SABER_TRY(full_mstep(c));
    if (par) return SABER_OK;
    c->stats.words_present = 0;
    for (const Chunk &ch : c->chunks) c->stats.words_present += ch.words_present;
    c->stats.light_tokens = c->T_light;
    return SABER_OK;
}

static int static_scratch_init(int device);

// Checks and sizes of saber_init_ex, or with `parent` of a context for held-out documents that borrows the parent's model.
static int make_ctx(saber_ctx **out, const int64_t *doc_ptr, const int32_t *word_ids, int64_t D, int32_t V,
                      int32_t K, float alpha, float beta, uint64_t seed, const saber_options *opt_in,
                      const saber_ctx *parent, bool no_state) {
    if (out) *out = nullptr;
    if (!out || !doc_ptr) return fail(SABER_EINVAL, "saber_init: null argument");
    if (D < 0 || V < 1 || K < 1) return fail(SABER_EINVAL, "saber_init: need D >= 0, V >= 1, K >= 1");
    if (!(alpha > 0.f) || !(beta > 0.f) || !std::isfinite(alpha) || !std::isfinite(beta))
        return fail(SABER_EINVAL, "saber_init: alpha and beta must be positive and finite");
    if (K > 262144) return fail(SABER_ERANGE, "saber_init: K = %d exceeds 262144 (three tree levels of width 64)", K);
    if (D > 0x7fffffffll) return fail(SABER_ERANGE, "saber_init: D exceeds 2^31 - 1");
    if (doc_ptr[0] != 0) return fail(SABER_EINVAL, "saber_init: doc_ptr[0] must be 0");
    int64_t maxlen = 0;
    for (int64_t d = 0; d < D; d++) {
        if (doc_ptr[d + 1] < doc_ptr[d]) return fail(SABER_EINVAL, "saber_init: doc_ptr decreases at document %lld", (long long)d);
        maxlen = std::max(maxlen, doc_ptr[d + 1] - doc_ptr[d]);
    }
    const int64_t T = doc_ptr[D];
    if (T >= (1ll << 40)) return fail(SABER_ERANGE, "saber_init: T = %lld tokens exceeds 2^40", (long long)T);
    if (T > 0 && !word_ids) return fail(SABER_EINVAL, "saber_init: word_ids is null");
    bool outside = false;   // (no way out of the loop: eight words at a time)
    for (int64_t t = 0; t < T; t++) outside |= (uint32_t)word_ids[t] >= (uint32_t)V;
    for (int64_t t = 0; outside && t < T; t++)
        if (word_ids[t] < 0 || word_ids[t] >= V)
            return fail(SABER_EINVAL, "saber_init: word id %d at token %lld is outside [0,%d)", word_ids[t], (long long)t, V);
    uint32_t bits = 1; while ((1u << bits) < (uint32_t)K) bits++;
    bool b16 = K <= 65536 && maxlen < 65536;   // the common case: topic and count both fit 16 bits
    if (b16) bits = 16;
    if (parent) { b16 = parent->b16; bits = parent->topic_bits; }   // the model's sparse rows of B fix the packing
    if (maxlen >= (1ll << (32 - bits)))
        return fail(SABER_ERANGE, "saber_init: longest document (%lld tokens) does not fit the %u count bits left by K = %d",
                    (long long)maxlen, 32 - bits, K);

    saber_options opt; saber_options_default(&opt);
    if (opt_in) {
        if (opt_in->n_chunks > 0) opt.n_chunks = opt_in->n_chunks;
        if (opt_in->block_threads > 0) opt.block_threads = opt_in->block_threads;
        if (opt_in->tile_tokens > 0) opt.tile_tokens = opt_in->tile_tokens;
        if (opt_in->long_doc_tokens > 0) opt.long_doc_tokens = opt_in->long_doc_tokens;
        if (opt_in->dz_lds_entries > 0) opt.dz_lds_entries = opt_in->dz_lds_entries;
        if (opt_in->stage_min_tokens > 0) opt.stage_min_tokens = opt_in->stage_min_tokens;
        if (opt_in->light_block_threads > 0) opt.light_block_threads = opt_in->light_block_threads;
        opt.light_word_tokens = opt_in->light_word_tokens;
        opt.stream_workers = opt_in->stream_workers;
        opt.ablation = opt_in->ablation;
        opt.device_mem_limit_mb = opt_in->device_mem_limit_mb;
        if (opt_in->quarter_row_entries != 0) opt.quarter_row_entries = std::max(0, opt_in->quarter_row_entries);
        if (opt_in->half_row_entries != 0) opt.half_row_entries = std::max(0, opt_in->half_row_entries);
        opt.stage_phi = opt_in->stage_phi; opt.profile = opt_in->profile;
        if (opt_in->stage_phi < 0) opt.stage_phi = 1;
    }
    if (opt.block_threads <= 0) opt.block_threads = 256;   // replaced below, once the LDS footprint is known
    if (opt.block_threads % 64 || opt.block_threads < 64 || opt.block_threads > 1024)
        return fail(SABER_EINVAL, "saber_init: block_threads must be a multiple of 64 in [64,1024]");
    if (opt.light_block_threads > 0 && (opt.light_block_threads % 64 || opt.light_block_threads > 1024))
        return fail(SABER_EINVAL, "saber_init: light_block_threads must be a multiple of 64 in [64,1024]");
    if (opt.stage_min_tokens <= 0) opt.stage_min_tokens = 1;
    if (opt.stream_workers < -1 || opt.stream_workers > kMaxSlots)
        return fail(SABER_EINVAL, "saber_init: stream_workers must be in [-1,%d]", kMaxSlots);
    if (parent) { opt.stream_workers = 0; opt.ablation = 0; }   // held-out documents are few: always resident, regular kernels
    if (opt.ablation < 0 || opt.ablation > 7 || (opt.ablation & 5) == 5)
        return fail(SABER_EINVAL, "saber_init: ablation must be in [0,7], and document order (bit 0) excludes alias tables (bit 2)");
    if (opt.ablation && opt.stream_workers) return fail(SABER_EINVAL, "saber_init: the ablation variants need stream_workers = 0");
    if (opt.ablation & 5) opt.light_word_tokens = -1;   // document order gathers Bhat from dense rows; alias tables are built from them
    if ((opt.ablation & 4) && alias_lds_bytes(K) > 159 * 1024)
        return fail(SABER_ERANGE, "saber_init: the alias-table variant needs 12 K bytes of LDS per workgroup, K = %d is beyond 13,500", K);
    const int32_t light_asked = opt.light_word_tokens;
    if (opt.light_word_tokens == 0) opt.light_word_tokens = std::max(1, K / 2);   // < 0 keeps every word dense
    // automatic: chunks of about 80 M tokens (T / 80 M, rounded to the nearest whole number).  The sampling pass of a
    // chunk reads every row of A of the chunk once per word of the document; at 0.4 to 0.7 non-zeros per token these rows
    // (4 bytes per entry) then fit the 256 MB Infinity Cache, and a corpus of several hundred million tokens samples
    // 20 % faster than in one chunk.  (Every chunk stages every word's Bhat row again: a 100 M-token corpus is fastest
    // in one chunk, and below 60 M tokens per chunk a large one slows down again.)
    if (opt.n_chunks <= 0) opt.n_chunks = (int32_t)std::max<int64_t>(1, (T + (40ll << 20)) / (80ll << 20));
    if (opt.n_chunks > 65536) return fail(SABER_EINVAL, "saber_init: n_chunks too large");
    if (opt.quarter_row_entries > 64 || opt.half_row_entries > 128)
        return fail(SABER_EINVAL, "saber_init: quarter_row_entries must not exceed 64 and half_row_entries 128");
    if (opt.dz_lds_entries > 12288) return fail(SABER_EINVAL, "saber_init: dz_lds_entries must not exceed 12288");
    // token positions inside a chunk are 32-bit: keep every chunk below 2^30 tokens (documents are far shorter)
    opt.n_chunks = (int32_t)std::max<int64_t>(opt.n_chunks, (T >> 30) + 1);
    if ((int64_t)opt.n_chunks > std::max<int64_t>(D, 1)) opt.n_chunks = (int32_t)std::max<int64_t>(D, 1);
    const int32_t tile_tokens_asked = opt.tile_tokens;

    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return fail(SABER_EDEVICE, "saber_init: no HIP device available");

    saber_ctx *c = new (std::nothrow) saber_ctx();
    if (!c) return fail(SABER_ENOMEM, "saber_init: out of host memory");
    c->hooks = parent ? parent->hooks : g_hooks;
    if (hipGetDevice(&c->device) != hipSuccess) { delete c; return fail(SABER_EDEVICE, "saber_init: hipGetDevice failed"); }
    { const int rc0 = static_scratch_init(c->device); if (rc0 != SABER_OK) { delete c; return rc0; } }
    c->D = D; c->T = T; c->V = V; c->K = K; c->alpha = alpha; c->beta = beta; c->seed = seed; c->opt = opt; c->tile_tokens_asked = tile_tokens_asked;
    c->parent = parent; c->no_state = no_state; c->max_doc_len = maxlen;
    c->n_slots = std::max(0, opt.stream_workers);
    c->Kpad = (K + 63) / 64 * 64;
    c->n3 = c->Kpad / 64;
    c->n3pad = (c->n3 + 63) / 64 * 64;
    c->b16 = b16;
    c->nwords = (K + 31) / 32;
    c->topic_bits = bits; c->count_bits = 32 - bits;
    c->pack = !b16 ? PACK_ANY : maxlen < (1 << 14) ? PACK_16_14 : PACK_16;   // (no count exceeds its document's length)
    c->z16 = K <= 65536;
    // the word's Bhat row is staged in LDS when it fits a workgroup's share: up to 150 KB of the CU's 160 KB
    if (hipDeviceGetAttribute(&c->lds_per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, 0) != hipSuccess || c->lds_per_cu <= 0)
        c->lds_per_cu = 64 * 1024;
    if (hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess || c->cus <= 0) c->cus = 256;
    const size_t stage_limit = std::min<size_t>(150 * 1024, (size_t)c->lds_per_cu > 10 * 1024 ? (size_t)c->lds_per_cu - 10 * 1024 : 0);
    c->staged = opt.stage_phi && estep_row_bytes(c) <= std::max<size_t>(stage_limit, 54 * 1024);
    const int64_t per_chunk = T / std::max(1, c->opt.n_chunks);
    // Rows too long for LDS: light words are read from memory with marks in LDS instead of from a full row in memory, whose
    // 4 K bytes per word would have to be written and read in every iteration.  An iteration (6 to 15) with all words dense and so:
    // T = 1.5 M, K = 70,000, V = 4,001 1.09 and 0.44 ms; 3 M, K = 45,000, V = 60,000 5.4 and 0.91; 20 M, V = 50,000 16.7 and 7.7.
    // In small chunks the longest words are cheaper with a dense row: counting a sparse one is the work of one workgroup
    // (T = 1.5 M: 0.50 ms with words of up to 32,768 tokens light, 0.44 with 8,192, 0.59 with 1,024; 20 M: 7.6, 8.4, 10.5).
    c->overlay = !c->staged && opt.stage_phi && opt.light_word_tokens > 0;
    if (c->overlay && light_asked == 0 && per_chunk < kLargeChunk) c->opt.light_word_tokens = std::min(c->opt.light_word_tokens, 8192);
    if (opt_in == nullptr || opt_in->block_threads <= 0) {
        c->opt.block_threads = estep_auto_block(c, per_chunk);
        c->auto_light_block = c->opt.light_block_threads <= 0;
    }
    if (c->opt.light_block_threads <= 0) c->opt.light_block_threads = c->opt.block_threads;
    // A part of LDS per sampling wavefront, where a CU still holds as many of them: an iteration at T = 2.3 M, K = 777 161 -> 149
    // us, T = 10 M, K = 1,000 583 -> 573, T = 100 K, K = 100 32.5 -> 31.5, T = 20 M, K = 2,000 (streamed, the link is the slower
    // one) 1,629 -> 1,628; T = 15 M, 370 tokens per document, K = 1,000 913 -> 890, 8,200 1,322 -> 1,304, 13,300 1,850 -> 1,820, 16,800
    // 1,620 -> 1,592, 30,000 2,382 -> 2,307; 94 tokens, K = 5,700 1,110 -> 1,087, 15,000 1,598 -> 1,551; T = 2 M, K = 300 to 37,030 0.2 to
    // 7 %.  Not for the sake of it: T = 36 M, K = 5,000 2.36 ms with 32 wavefronts per CU and lane
    // permutations, 2.51 with 24 of the same workgroups, 2.62 with 32 in larger ones; T = 100 M, K = 10,000 7.1 and 7.4.  Of chunks
    // of 4 M tokens and more it is in use at K up to 1,048, from 1,221 to 2,104, 2,733 to 4,216, 5,665 to 5,792, 6,613 to 8,440, 10,077 to 11,588,
    // 13,229 to 16,884 and 20,161 to 37,048.
    // (The kernel is built for the packing of counts below 2^14 only; what it exchanges would be the same for the others.)
    if (c->staged && c->z16 && c->pack == PACK_16_14) {
        const int without = estep_waves_per_cu(c, c->opt.block_threads, kLdsPiece), light = estep_waves_per_cu(c, c->opt.light_block_threads, kLdsPiece);
        c->slots = true;
        c->slots = estep_waves_per_cu(c, c->opt.block_threads, kLdsPiece) == without && estep_waves_per_cu(c, c->opt.light_block_threads, kLdsPiece) == light;
    }
    if (c->opt.tile_tokens <= 0) c->opt.tile_tokens = auto_tile_tokens(c, per_chunk);
    c->vbeta = (float)V * beta;
    int rc = check_estep_lds_layout<PACK_16>();
    if (rc == SABER_OK) rc = check_estep_lds_layout<PACK_16_14>();
    if (rc != SABER_OK) { delete c; return rc; }
    *out = c;
    return SABER_OK;
}

extern "C" int saber_init_ex(saber_ctx **out, const int64_t *doc_ptr, const int32_t *word_ids, int64_t D, int32_t V,
                             int32_t K, float alpha, float beta, uint64_t seed, const saber_options *opt_in) {
    if (!out) return fail(SABER_EINVAL, "saber_init: null argument");
    saber_ctx *c = nullptr;
    *out = nullptr;
    int rc = make_ctx(&c, doc_ptr, word_ids, D, V, K, alpha, beta, seed, opt_in, nullptr, false);
    if (rc != SABER_OK) return rc;
    try {
        Layout lay;
        rc = lay_out(c, doc_ptr, word_ids, lay);
        if (rc == SABER_OK) rc = upload(c, doc_ptr, word_ids, lay);
    } catch (const std::bad_alloc &) { rc = fail(SABER_ENOMEM, "saber_init: out of host memory"); }
    if (rc != SABER_OK) { saber_free(c); return rc; }
    *out = c;
    return SABER_OK;
}

extern "C" int saber_init(saber_ctx **out, const int64_t *doc_ptr, const int32_t *word_ids, int64_t D, int32_t V,
                          int32_t K, float alpha, float beta, uint64_t seed) {
    return saber_init_ex(out, doc_ptr, word_ids, D, V, K, alpha, beta, seed, nullptr);
}

// ------------------------------------------------------------------------------------------------
// saber_iterate
// ------------------------------------------------------------------------------------------------
extern "C" int saber_iterate(saber_ctx *c, int32_t n) {
    if (!c) return fail(SABER_EINVAL, "saber_iterate: null context");
    if (n < 0) return fail(SABER_EINVAL, "saber_iterate: n must be >= 0");
    const bool prof = c->opt.profile != 0;
    int32_t done = 0;
    while (done < n) {
        const int batch = std::min<int32_t>(n - done, kMaxTimedIters);
        // per-iteration device counters: {dense-branch tokens, nnz(A), sum_d K_d L_d}
        hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, c->stream, (uint32_t *)c->counters, 0u,
                           (size_t)kMaxTimedIters * kCtr * 2);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for((int64_t)batch * kDenseSlots * 2, 256)), dim3(256), 0, c->stream,
                           (uint32_t *)c->dense_slots, 0u, (size_t)batch * kDenseSlots * 2);
        HIP_TRY(hipGetLastError());
        for (int b = 0; b < batch; b++) {
            hipEvent_t *ev = c->ev + (size_t)b * EV_PER_ITER;
            c->iter++;
            if (prof) HIP_TRY(hipEventRecord(ev[EV_BEGIN], c->stream));
            // E-step: z <- Sample(A_d, Bhat_v, Q_v, T_v) for every token, written in document order and in word order
            if (c->opt.ablation & 1) SABER_TRY(launch_estep_docmajor(c, c->dense_slots + (size_t)kDenseSlots * b));
            else for (const Chunk &ch : c->chunks) {
                int s = -1;
                if (c->n_slots) SABER_TRY(stream_acquire(c, ch, &s));
                EStepParams p = make_params(c, ch, s);
                p.n_dense = c->dense_slots + (size_t)kDenseSlots * b;
                SABER_TRY(launch_estep<MODE_SAMPLE>(c, c, ch, p));
                if (c->n_slots) {
                    // the chunk's rows of A are rebuilt while its new assignments are in the buffer (the sampling
                    // of later chunks reads other documents' rows only); after that only z_wm keeps them
                    SABER_TRY(launch_count_dz_chunk(c, ch, s));
                    SABER_TRY(stream_release(c, s));
                }
            }
            if (prof) HIP_TRY(hipEventRecord(ev[EV_SAMPLE], c->stream));
            // M-step
            const unsigned long long *slots = c->dense_slots + (size_t)kDenseSlots * b;
            if (c->joined) {
                SABER_TRY(launch_joined_mstep(c, slots, c->counters + kCtr * b, prof ? ev[EV_DZ] : nullptr));
                if (prof) HIP_TRY(hipEventRecord(ev[EV_PHI], c->stream));   // (no EV_CK: the totals are counted with the rest)
                continue;
            }
            if (c->n_slots) SABER_TRY(launch_segmented_count(c, SegLists{}, own_light_segments(c)));
            else SABER_TRY(launch_counts(c));
            if (prof) HIP_TRY(hipEventRecord(ev[EV_DZ], c->stream));
            SABER_TRY(launch_count_slabs(c, c->n_vz_long, true));
            if (prof) HIP_TRY(hipEventRecord(ev[EV_CK], c->stream));
            SABER_TRY(launch_phi(c));
            SABER_TRY(launch_light_words(c));
            if (prof) HIP_TRY(hipEventRecord(ev[EV_PHI], c->stream));
            SABER_TRY(launch_stats(c, slots, c->counters + kCtr * b));
        }
        SABER_TRY(sync_all(c));
        unsigned long long h[kMaxTimedIters * kCtr];
        HIP_TRY(hipMemcpy(h, c->counters, sizeof(h), hipMemcpyDeviceToHost));
        for (int b = 0; b < batch; b++) {
            // the E-step of this iteration read the rows counted at the end of the previous one
            c->stats.sum_tokens += c->T;
            c->stats.sum_tokens_dense += (int64_t)h[kCtr * b];
            c->stats.sum_row_entries += c->stats.next_row_entries;
            c->stats.sum_row_fetch += c->stats.next_row_fetch;
            c->stats.sum_light_entries += c->stats.next_light_entries;
            c->stats.nnz_cd = (int64_t)h[kCtr * b + 1];
            c->stats.next_row_entries = (int64_t)h[kCtr * b + 2];
            c->stats.next_row_fetch = (int64_t)h[kCtr * b + 3];
            c->stats.next_light_entries = (int64_t)h[kCtr * b + 4];
            if (prof) {
                hipEvent_t *ev = c->ev + (size_t)b * EV_PER_ITER;
                float ms[4] = {}, tot;
                for (int s = 0; s < 4; s++) {
                    if (s == EV_DZ && c->joined) continue;
                    HIP_TRY(hipEventElapsedTime(&ms[s], ev[s == EV_CK && c->joined ? EV_DZ : s], ev[s + 1]));
                }
                HIP_TRY(hipEventElapsedTime(&tot, ev[EV_BEGIN], ev[EV_PHI]));
                c->stats.ms_sample += ms[0]; c->stats.ms_count_dz += ms[1]; c->stats.ms_ck += ms[2];
                c->stats.ms_phi += ms[3]; c->stats.ms_total += tot;
                c->stats.sample_launches += (int64_t)c->chunks.size();
            }
            c->stats.iterations++;
        }
        done += batch;
    }
    return SABER_OK;
}

// ------------------------------------------------------------------------------------------------
// outputs
// ------------------------------------------------------------------------------------------------
// Makes a device current for a scope; the one that was current before comes back at its end.
struct DeviceScope {
    int before = -1;
    explicit DeviceScope(int device) {
        int now = device;
        if (hipGetDevice(&now) == hipSuccess && now != device && hipSetDevice(device) == hipSuccess) before = now;
    }
    ~DeviceScope() { if (before >= 0) (void)hipSetDevice(before); }
};

// Whether so many bytes for the caller are worth threads, and the bytes of the pieces they are cut into (a longer row is a
// piece of its own).
static bool pull_many(const saber_ctx *c, int64_t out_bytes, PullBy by) {
    return out_bytes > (c->staging.bytes >= (size_t)(kPullSlots / 2 * kPullPiece) ? by.next : by.many);
}
static int64_t pull_piece(bool many) { return many ? kPullPiece : kPullPiece / 4; }

// Results on their way to the caller's memory: piece i, the elements [cuts[i], cuts[i + 1]) of the device array, is handed
// to consume(i, host pointer), which puts it where it belongs.  How that is done depends on the bytes written for the caller
// (out_bytes):
//   * above by.many, or by.next, by way of pinned staging of kPullSlots slots, which up to kPullThreads threads consume while
//     the next pieces are in flight.  A caller's fresh pages cost far more than the link: into ordinary memory a copy of
//     100 M assignments as int32 took 44 ms, as 16 bits through this path 8;
//   * below, the calling thread alone, out of two small slots: threads, and the first touch of pinned memory, cost a
//     context's first call a millisecond (A in CSR of T = 1 M, K = 100, first and later calls: 1.62 and 0.25 ms with them,
//     0.36 and 0.34 this way, 0.45 and 0.41 by a plain copy);
//   * up to by.few by plain copies into ordinary memory (the assignments of T = 300,000: 0.07 and 0.05 ms, 0.24 and 0.06
//     through two slots; 4 MB of rows of B: 0.23 ms, 0.36 through two slots, 0.29 with threads - which are the faster ones by
//     0.2 ms for 3.5 MB after 20 MB of A).  consume() hides under no copy then, so that is less where it takes entries apart.
// The threads end before the call returns; consume must not throw.  No piece may exceed kPullPiece bytes.
// Events belong to the device that is current when they are made, and only its streams record them; the caller may have
// another one current.
template <typename F>
static int pull(saber_ctx *c, const void *dev, size_t elem, const std::vector<int64_t> &cuts, int64_t out_bytes, PullBy by, F consume) {
    const int64_t np = (int64_t)cuts.size() - 1;
    if (np <= 0) return SABER_OK;
    auto piece_bytes = [&](int64_t k) { return (size_t)(cuts[(size_t)k + 1] - cuts[(size_t)k]) * elem; };
    auto source = [&](int64_t k) { return (const char *)dev + (size_t)cuts[(size_t)k] * elem; };
    size_t largest = 1;
    for (int64_t i = 0; i < np; i++) largest = std::max(largest, piece_bytes(i));
    const bool many = pull_many(c, out_bytes, by);
    if (out_bytes <= by.few && !many) {
        const int64_t group = kPullPiece / (int64_t)elem;   // as many pieces at a time as that
        const std::unique_ptr<char[]> host(new char[std::max(largest, (size_t)std::min(cuts.back(), group) * elem)]);
        HIP_TRY(hipStreamSynchronize(c->stream));
        for (int64_t k = 0, end; k < np; k = end) {
            for (end = k + 1; end < np && cuts[(size_t)end + 1] - cuts[(size_t)k] <= group;) end++;
            const size_t bytes = (size_t)(cuts[(size_t)end] - cuts[(size_t)k]) * elem;
            if (bytes) HIP_TRY(hipMemcpy(host.get(), source(k), bytes, hipMemcpyDeviceToHost));
            for (int64_t i = k; i < end; i++) consume(i, (const void *)(host.get() + (size_t)(cuts[(size_t)i] - cuts[(size_t)k]) * elem));
        }
        return SABER_OK;
    }
    const DeviceScope scope(c->device);
    if (!many) largest = std::max(largest, (size_t)pull_piece(many));   // (so that the slots serve later calls as well)
    largest = (largest + 255) & ~(size_t)255;
    const int slots = many ? (int)std::min<int64_t>(np, kPullSlots) : 2;
    if (c->staging.bytes < largest * (size_t)slots) {
        if (c->staging.buf) { if (c->staging.pinned) (void)hipHostFree(c->staging.buf); else free(c->staging.buf); }
        c->staging.buf = nullptr; c->staging.bytes = 0; c->staging.pinned = true;
        if (hipHostMalloc((void **)&c->staging.buf, largest * (size_t)slots, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            c->staging.pinned = false;
            c->staging.buf = (char *)malloc(largest * (size_t)slots);
            if (!c->staging.buf) return fail(SABER_ENOMEM, "out of host memory");
        }
        c->staging.bytes = largest * (size_t)slots;
    }
    for (int i = 0; i < slots; i++)
        if (!c->staging.ev[i]) HIP_TRY(hipEventCreateWithFlags(&c->staging.ev[i], hipEventDisableTiming));
    auto slot = [&](int64_t k) { return c->staging.buf + (size_t)(k % slots) * largest; };
    auto request = [&](int64_t k) {
        hipError_t e = hipSuccess;
        if (piece_bytes(k)) e = hipMemcpyAsync(slot(k), source(k), piece_bytes(k), hipMemcpyDeviceToHost, c->stream);
        if (e == hipSuccess) e = hipEventRecord(c->staging.ev[k % slots], c->stream);
        return e;
    };
    std::vector<std::atomic<char>> done(many ? (size_t)np : 0);
    for (auto &d : done) d.store(0, std::memory_order_relaxed);
    std::atomic<int64_t> issued{0}, next{0};
    std::atomic<int> error{(int)hipSuccess};
    auto work = [&]() {
        (void)hipSetDevice(c->device);
        for (;;) {
            const int64_t k = next.fetch_add(1);
            if (k >= np) return;
            while (issued.load(std::memory_order_acquire) <= k) {
                if (error.load() != (int)hipSuccess) return;
                std::this_thread::yield();
            }
            const hipError_t e = hipEventSynchronize(c->staging.ev[k % slots]);
            if (e != hipSuccess) { error.store((int)e); return; }
            consume(k, (const void *)slot(k));
            done[(size_t)k].store(1, std::memory_order_release);
        }
    };
    std::vector<std::thread> threads;
    if (many && np > 2) {
        try {
            threads.reserve(kPullThreads);
            for (int64_t i = 0; i < std::min<int64_t>(np, kPullThreads); i++) threads.emplace_back(work);
        } catch (...) {}   // with fewer threads, or none, it only takes longer
    }
    hipError_t e = hipSuccess;
    if (threads.empty()) {
        if (slots > 1) e = request(0);
        for (int64_t k = 0; k < np && e == hipSuccess; k++) {   // piece k + 1 goes to the other slot, free since piece k - 1
            if (slots == 1) e = request(k);
            else if (k + 1 < np) e = request(k + 1);
            if (e == hipSuccess) e = hipEventSynchronize(c->staging.ev[k % slots]);
            if (e == hipSuccess) consume(k, (const void *)slot(k));
        }
    }
    for (int64_t k = 0; k < np && !threads.empty(); k++) {
        while (k >= slots && !done[(size_t)(k - slots)].load(std::memory_order_acquire) && error.load() == (int)hipSuccess)
            std::this_thread::yield();
        if (error.load() != (int)hipSuccess) break;
        e = request(k);
        if (e != hipSuccess) break;
        issued.store(k + 1, std::memory_order_release);
    }
    if (e != hipSuccess) error.store((int)e);
    for (auto &t : threads) t.join();
    e = (hipError_t)error.load();
    if (e != hipSuccess) return fail(SABER_EDEVICE, "copying results from the device failed: %s", hipGetErrorString(e));
    return SABER_OK;
}

// n assignments from the device array z (of the context's assignment type) to the caller's int32
static int pull_z(saber_ctx *c, const void *z, int64_t n, int32_t *out) {
    const int64_t elem = c->z16 ? 2 : 4;
    if (!c->z16 && n * elem <= kPullZ.many) {   // nothing to convert: straight to the caller's memory
        HIP_TRY(hipStreamSynchronize(c->stream));
        HIP_TRY(hipMemcpy(out, z, (size_t)n * 4, hipMemcpyDeviceToHost));
        return SABER_OK;
    }
    // (pieces of a sixteenth of the array, 128 K to 512 K assignments: a small one is shared by the threads as well)
    const int64_t piece = std::min<int64_t>(kPullPiece / elem, std::max<int64_t>(131072, (n / 16 + 4095) & ~4095ll));
    std::vector<int64_t> cuts(1, 0);
    while (cuts.back() < n) cuts.push_back(std::min<int64_t>(n, cuts.back() + piece));
    return pull(c, z, (size_t)elem, cuts, n * 4, kPullZ, [&](int64_t i, const void *host) {
        const int64_t a = cuts[(size_t)i], m = cuts[(size_t)i + 1] - a;
        if (elem == 4) { memcpy(out + a, host, (size_t)m * 4); return; }
        const uint16_t *src = (const uint16_t *)host;
        for (int64_t j = 0; j < m; j++) out[a + j] = (int32_t)src[j];
    });
}

extern "C" int saber_counts_nnz(saber_ctx *c, int64_t *nnz) {
    if (!c || !nnz) return fail(SABER_EINVAL, "saber_counts_nnz: null argument");
    try {
        std::vector<uint2> rec((size_t)c->D);
        if (c->D) HIP_TRY(hipMemcpy(rec.data(), c->docrec, sizeof(uint2) * (size_t)c->D, hipMemcpyDeviceToHost));
        int64_t s = 0; for (auto &r : rec) s += r.y;
        *nnz = s;
    } catch (const std::bad_alloc &) { return fail(SABER_ENOMEM, "saber_counts_nnz: out of host memory"); }
    return SABER_OK;
}

extern "C" int saber_counts(saber_ctx *c, int64_t *cd_row_ptr, int32_t *cd_topic, int32_t *cd_count, int32_t *cwk,
                            int64_t *ck) {
    if (!c) return fail(SABER_EINVAL, "saber_counts: null context");
    if ((cd_topic || cd_count) && !cd_row_ptr) return fail(SABER_EINVAL, "saber_counts: cd_topic/cd_count need cd_row_ptr");
    const uint32_t cmask = (1u << c->count_bits) - 1u;
    try {
        if (cd_row_ptr) {
            std::vector<uint2> rec((size_t)c->D);
            if (c->D) HIP_TRY(hipMemcpy(rec.data(), c->docrec, sizeof(uint2) * (size_t)c->D, hipMemcpyDeviceToHost));
            cd_row_ptr[0] = 0;
            for (int64_t d = 0; d < c->D; d++) cd_row_ptr[d + 1] = cd_row_ptr[d] + rec[(size_t)d].y;
            if (cd_topic || cd_count) {
                // unpack the device rows by pieces of whole documents (format conversion only)
                std::vector<int64_t> cuts(1, 0), piece_doc(1, 0);
                const int64_t out_bytes = 4 * std::max(2 * cd_row_ptr[c->D], c->cd_cap);
                const int64_t piece = pull_piece(pull_many(c, out_bytes, kPullEntries));
                for (int64_t d = 0; d < c->D; d++) {
                    const int64_t end = d + 1 < c->D ? (int64_t)rec[(size_t)d + 1].x * 32 : c->cd_cap;
                    if ((end - cuts.back()) * 4 > piece) { cuts.push_back((int64_t)rec[(size_t)d].x * 32); piece_doc.push_back(d); }
                }
                cuts.push_back(c->cd_cap); piece_doc.push_back(c->D);
                SABER_TRY(pull(c, c->cd_ent, sizeof(uint32_t), cuts, out_bytes, kPullEntries, [&](int64_t i, const void *host) {
                    for (int64_t d = piece_doc[(size_t)i]; d < piece_doc[(size_t)i + 1]; d++) {
                        const uint32_t *row = (const uint32_t *)host + ((int64_t)rec[(size_t)d].x * 32 - cuts[(size_t)i]);
                        int64_t o = cd_row_ptr[d];
                        for (uint32_t j = 0; j < rec[(size_t)d].y; j++, o++) {
                            if (cd_topic) cd_topic[o] = (int32_t)(row[j] >> c->count_bits);
                            if (cd_count) cd_count[o] = (int32_t)(row[j] & cmask);
                        }
                    }
                }));
            }
        }
        if (cwk) {
            // dense rows: B is consumed (and cleared) by the Bhat kernel; rebuild it from z for export
            if (c->V_dense) {
                std::vector<int32_t> row_word((size_t)c->V_dense + 1);
                HIP_TRY(hipMemcpy(row_word.data(), c->row_word, sizeof(int32_t) * row_word.size(), hipMemcpyDeviceToHost));
                const int64_t out_bytes = 4 * (int64_t)c->V_dense * c->Kpad;
                const int64_t piece = pull_piece(pull_many(c, out_bytes, kPullRows));
                const int64_t rows = std::max<int64_t>(1, piece / ((int64_t)c->Kpad * 4));   // (Kpad * 4 is at most 1 MB)
                std::vector<int64_t> cuts(1, 0);
                while (cuts.back() < (int64_t)c->V_dense * c->Kpad)
                    cuts.push_back(std::min<int64_t>((int64_t)c->V_dense * c->Kpad, cuts.back() + rows * c->Kpad));
                SABER_TRY(launch_count_slabs(c, c->n_vz_items, false));
                SABER_TRY(pull(c, c->cwk, sizeof(int32_t), cuts, out_bytes, kPullRows, [&](int64_t i, const void *host) {
                    for (int64_t e = cuts[(size_t)i]; e < cuts[(size_t)i + 1]; e += c->Kpad)
                        memcpy(cwk + (size_t)row_word[(size_t)(e / c->Kpad)] * (size_t)c->K, (const int32_t *)host + (e - cuts[(size_t)i]),
                               sizeof(int32_t) * (size_t)c->K);
                }));
                SABER_TRY(launch_clear_accumulators(c, false));   // (an export that broke off leaves that to the next count)
                HIP_TRY(hipStreamSynchronize(c->stream));
            }
            // light words: unpack the sparse rows by pieces of whole words (format conversion only)
            if (c->V_light) {
                std::vector<uint2> by_number((size_t)c->V_light), wrec((size_t)c->V_light);   // by number; as the rows lie, like lwords
                std::vector<int32_t> lwords((size_t)c->V_light);
                HIP_TRY(hipMemcpy(by_number.data(), c->wrec, sizeof(uint2) * by_number.size(), hipMemcpyDeviceToHost));
                size_t n = 0;
                for (int32_t v = 0; v < c->V; v++) {
                    const int32_t row = c->h_word_row[(size_t)v];
                    if (row < 0) { lwords[n] = v; wrec[n++] = by_number[(size_t)(-row - 1)]; }
                }
                std::vector<int64_t> cuts(1, 0), piece_word(1, 0);
                // (a word's row of K counts has to be cleared as well: threads share those out by at most 1 MB per piece)
                const int64_t out_bytes = 4 * std::max((int64_t)c->V_light * c->K, c->lw_cap);
                const bool many = pull_many(c, out_bytes, kPullRows);
                const int64_t piece = pull_piece(many), most = many ? std::max<int64_t>(1, kPullPiece / (4 * (int64_t)c->K)) : c->V_light;
                for (int64_t li = 0; li < c->V_light; li++) {
                    const int64_t end = li + 1 < c->V_light ? (int64_t)wrec[(size_t)li + 1].x * 32 : c->lw_cap;
                    if ((end - cuts.back()) * 4 > piece || li - piece_word.back() >= most) {
                        cuts.push_back((int64_t)wrec[(size_t)li].x * 32); piece_word.push_back(li);
                    }
                }
                cuts.push_back(c->lw_cap); piece_word.push_back(c->V_light);
                SABER_TRY(pull(c, c->lw_ent, sizeof(uint32_t), cuts, out_bytes, kPullRows, [&](int64_t i, const void *host) {
                    for (int64_t li = piece_word[(size_t)i]; li < piece_word[(size_t)i + 1]; li++) {
                        int32_t *row = cwk + (size_t)lwords[(size_t)li] * (size_t)c->K;
                        memset(row, 0, sizeof(int32_t) * (size_t)c->K);
                        const uint32_t *e = (const uint32_t *)host + ((int64_t)wrec[(size_t)li].x * 32 - cuts[(size_t)i]);
                        for (uint32_t j = 0; j < wrec[(size_t)li].y; j++) row[e[j] >> c->count_bits] = (int32_t)(e[j] & cmask);
                    }
                }));
            }
        }
        if (ck) {
            std::vector<unsigned long long> h((size_t)c->K);
            HIP_TRY(hipMemcpy(h.data(), c->ck, sizeof(unsigned long long) * (size_t)c->K, hipMemcpyDeviceToHost));
            for (int32_t k = 0; k < c->K; k++) ck[k] = (int64_t)h[(size_t)k];
        }
    } catch (const std::bad_alloc &) { return fail(SABER_ENOMEM, "saber_counts: out of host memory"); }
    return SABER_OK;
}

// *result (device memory) = [ sum over the tokens of c of ln(S_t + Q_w)  -  sum_d w_d ln(len_d + K alpha) ] / T on the device, all
// sums in binary64 and in a fixed order.  `theta` holds the rows of A that S is formed with (c itself for the training
// log-likelihood; the observed part of the documents for the holdout score, whose document lengths then also give
// len_d while w_d counts the scored tokens).  Everything is queued on c's stream; nothing is waited for.
static int launch_loglik(saber_ctx *c, const saber_ctx *theta, const LlScratch &ws, double *result) {
    bool first = true;
    for (const Chunk &ch : c->chunks) {
        if (ch.ntiles == 0) continue;
        int s = -1;
        if (c->n_slots) SABER_TRY(stream_acquire(c, ch, &s));
        EStepParams p = make_params(c, ch, s);
        p.out_ll = ws.tile_part;
        SABER_TRY(launch_estep<MODE_LOGLIK>(c, theta, ch, p));
        if (c->n_slots) SABER_TRY(stream_release(c, s));
        hipLaunchKernelGGL(reduce_partials_kernel, dim3(kReduceBlocks), dim3(kReduceThreads), 0, c->stream, ws.tile_part,
                           ch.ntiles, ws.block_part);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(kReduceThreads), 0, c->stream, ws.block_part, ws.acc, first ? 0 : 1);
        HIP_TRY(hipGetLastError());
        first = false;
    }
    hipLaunchKernelGGL(doc_norm_kernel, dim3(kReduceBlocks), dim3(kReduceThreads), 0, c->stream, c->doc_ptr, theta->doc_ptr,
                       c->D, (double)c->K * (double)c->alpha, ws.block_part);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(kReduceThreads), 0, c->stream, ws.block_part, ws.norm, 0);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(loglik_finish_kernel, dim3(1), dim3(64), 0, c->stream, ws.acc, ws.norm, (double)c->T, result);
    HIP_TRY(hipGetLastError());
    return SABER_OK;
}

extern "C" int saber_loglik(saber_ctx *c, double *out) {
    if (!c || !out) return fail(SABER_EINVAL, "saber_loglik: null argument");
    if (c->T == 0) { *out = 0.0; return SABER_OK; }
    const LlScratch ws = ll_scratch(c->ll_partial, (size_t)std::max<int64_t>(c->max_chunk_tiles, 1));
    SABER_TRY(launch_loglik(c, c, ws, ws.result));
    SABER_TRY(sync_all(c));
    HIP_TRY(hipMemcpy(out, ws.result, sizeof(double), hipMemcpyDeviceToHost));
    return SABER_OK;
}

// ---- the same reduction for callers that must not allocate ----
// The work space is a file-scope device array instead of the context's allocation.  Every device has its own copy of
// the array at its own address, looked up once per device (saber_init does it, with that device current); host code
// uses that address only, never the array's name.
constexpr size_t kStaticLlTiles = (size_t)1 << 20;   // per-tile sums of one chunk: 8 MB
constexpr int kMaxDevices = 64;
static __device__ __align__(256) double g_ll_static[kStaticLlTiles + kLlTail];
static double *g_ll_static_ptr[kMaxDevices] = {};

static int static_scratch_init(int device) {
    if (device < 0 || device >= kMaxDevices) return fail(SABER_ERANGE, "device %d is beyond the %d devices the library keeps work space for", device, kMaxDevices);
    if (g_ll_static_ptr[device]) return SABER_OK;
    double *ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(g_ll_static)));
    if (!ptr) return fail(SABER_EDEVICE, "hipGetSymbolAddress returned no address for the static work space");
    g_ll_static_ptr[device] = ptr;
    return SABER_OK;
}

extern "C" int saber_loglik_static(saber_ctx *c, double *d_result) {
    if (!c || !d_result) return fail(SABER_EINVAL, "saber_loglik_static: null argument");
    if ((size_t)c->max_chunk_tiles > kStaticLlTiles)
        return fail(SABER_ERANGE, "saber_loglik_static: a chunk of %lld sampling workgroups exceeds the static work space of %zu "
                    "(use saber_loglik, or more chunks)", (long long)c->max_chunk_tiles, kStaticLlTiles);
    double *base = (c->device >= 0 && c->device < kMaxDevices) ? g_ll_static_ptr[c->device] : nullptr;
    if (!base) return fail(SABER_ESTATE, "saber_loglik_static: no static work space on device %d", c->device);
    if (c->T == 0) {
        hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, c->stream, reinterpret_cast<uint32_t *>(d_result), 0u, (size_t)2);
        HIP_TRY(hipGetLastError());
    } else {
        SABER_TRY(launch_loglik(c, c, ll_scratch(base, kStaticLlTiles), d_result));
    }
    return sync_all(c);
}

// ------------------------------------------------------------------------------------------------
// holdout log-likelihood (document completion on held-out documents, model frozen)
// ------------------------------------------------------------------------------------------------
// n E-steps + CountByDZ on a context that borrows a model: Alg. 1 restricted to A
static int foldin_iterate(saber_ctx *c, int32_t n) {
    for (int32_t i = 0; i < n; i++) {
        c->iter++;
        hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for((int64_t)kDenseSlots * 2, 256)), dim3(256), 0, c->stream,
                           (uint32_t *)c->dense_slots, 0u, (size_t)kDenseSlots * 2);
        HIP_TRY(hipGetLastError());
        for (const Chunk &ch : c->chunks) {
            EStepParams p = make_params(c, ch);
            p.n_dense = c->dense_slots;
            SABER_TRY(launch_estep<MODE_SAMPLE>(c, c, ch, p));
        }
        SABER_TRY(launch_counts(c));
    }
    HIP_TRY(hipStreamSynchronize(c->stream));
    return SABER_OK;
}

// lay_out() of a context on a trained model by another thread where that pays (1.5 ms for the 550,000 scored tokens of 3,300
// documents, which the observed ones' layout and fold-in hide; a thread costs 0.03); by the calling one at finish() otherwise.
struct BackgroundLayout {
    Layout lay;
    std::thread thread;
    int rc = SABER_OK;
    bool no_memory = false;
    std::string error;
    void run(saber_ctx *c, const int64_t *doc_ptr, const int32_t *word_ids) {
        try {
            rc = lay_out(c, doc_ptr, word_ids, lay);
            if (rc != SABER_OK) error = g_err;
        } catch (const std::bad_alloc &) { rc = SABER_ENOMEM; no_memory = true; }
    }
    void start(saber_ctx *c, const int64_t *doc_ptr, const int32_t *word_ids) {
        if (c->T < 32768) return;
        try { thread = std::thread([=] { run(c, doc_ptr, word_ids); }); } catch (const std::system_error &) {}   // no thread to be had
    }
    int finish(saber_ctx *c, const int64_t *doc_ptr, const int32_t *word_ids) {
        if (thread.joinable()) thread.join(); else run(c, doc_ptr, word_ids);
        return rc == SABER_OK ? rc : fail(rc, "%s", no_memory ? "saber_holdout_loglik: out of host memory" : error.c_str());
    }
    ~BackgroundLayout() { if (thread.joinable()) thread.join(); }
};

// The checked call.  *no_memory: host memory ran out.
static int holdout_loglik(saber_ctx *m, const int64_t *doc_ptr, const int32_t *word_ids, const uint8_t *observed, int64_t D,
                          int32_t n_foldin, uint64_t seed, const int32_t *z_init, int32_t *z_out, double *loglik, int64_t *n_scored,
                          bool side_by_side, bool *no_memory) {
    const int64_t T = doc_ptr[D];
    saber_ctx *obs = nullptr, *scr = nullptr;
    int rc = SABER_OK;
    *no_memory = false;
    try {
        // the observed part and the scored part as two corpora over the same documents (every word is written to both and one
        // of the two positions moves on: which one cannot be foretold)
        std::vector<int64_t> optr((size_t)D + 1, 0), sptr((size_t)D + 1, 0);
        for (int64_t d = 0; d < D; d++) {
            int64_t n = 0;
            for (int64_t t = doc_ptr[d]; t < doc_ptr[d + 1]; t++) n += observed[t] != 0;
            optr[(size_t)d + 1] = optr[(size_t)d] + n; sptr[(size_t)d + 1] = doc_ptr[d + 1] - optr[(size_t)d + 1];
        }
        std::vector<int32_t> ow((size_t)optr[(size_t)D] + 1), sw((size_t)sptr[(size_t)D] + 1);
        int32_t *po = ow.data(), *ps = sw.data();
        for (int64_t t = 0; t < T; t++) {
            const bool o = observed[t] != 0;
            *po = *ps = word_ids[t];
            po += o; ps += !o;
        }
        saber_options opt = m->opt;
        opt.profile = 0; opt.n_chunks = 1; opt.tile_tokens = m->tile_tokens_asked;   // (0: sized for these documents)
        if (m->auto_light_block) opt.block_threads = opt.light_block_threads = 0;
        rc = make_ctx(&obs, optr.data(), ow.data(), D, m->V, m->K, m->alpha, m->beta, seed, &opt, m, false);
        if (rc == SABER_OK) rc = make_ctx(&scr, sptr.data(), sw.data(), D, m->V, m->K, m->alpha, m->beta, seed, &opt, m, true);
        BackgroundLayout scr_lay;
        if (rc == SABER_OK && side_by_side) scr_lay.start(scr, sptr.data(), sw.data());
        if (rc == SABER_OK) {
            Layout lay;
            rc = lay_out(obs, optr.data(), ow.data(), lay);
            if (rc == SABER_OK) rc = upload(obs, optr.data(), ow.data(), lay);
        }
        if (rc == SABER_OK && z_init) rc = saber_set_z(obs, z_init, 0);
        if (rc == SABER_OK) rc = foldin_iterate(obs, n_foldin);
        if (rc == SABER_OK && z_out) {
            // the model's, which outlives the call (its events are of the model's device)
            const bool borrow = obs->device == m->device;
            if (borrow) std::swap(obs->staging, m->staging);
            rc = saber_get_z(obs, z_out);
            if (borrow) std::swap(obs->staging, m->staging);
        }
        if (rc == SABER_OK) { rc = scr_lay.finish(scr, sptr.data(), sw.data()); *no_memory = scr_lay.no_memory; }
        if (rc == SABER_OK) rc = upload(scr, sptr.data(), sw.data(), scr_lay.lay);
        double ll = 0.0;
        if (rc == SABER_OK && scr->T > 0) {
            // theta comes from the observed part: its rows of A, and its document lengths in the normaliser
            const LlScratch ws = ll_scratch(scr->ll_partial, (size_t)std::max<int64_t>(scr->max_chunk_tiles, 1));
            rc = launch_loglik(scr, obs, ws, ws.result);
            if (rc == SABER_OK) {
                hipError_t e = hipStreamSynchronize(scr->stream);
                if (e == hipSuccess) e = hipMemcpy(&ll, ws.result, sizeof(double), hipMemcpyDeviceToHost);
                if (e != hipSuccess) rc = fail(SABER_EDEVICE, "saber_holdout_loglik: %s", hipGetErrorString(e));
            }
        }
        if (rc == SABER_OK) {
            *n_scored = scr->T;
            *loglik = ll;
        }
    } catch (const std::bad_alloc &) { rc = fail(SABER_ENOMEM, "saber_holdout_loglik: out of host memory"); *no_memory = true; }
    saber_free(scr); saber_free(obs);
    return rc;
}

extern "C" int saber_holdout_loglik(saber_ctx *m, const int64_t *doc_ptr, const int32_t *word_ids,
                                    const uint8_t *observed, int64_t D, int32_t n_foldin, uint64_t seed,
                                    const int32_t *z_init, int32_t *z_out, double *loglik, int64_t *n_scored) {
    if (!m || !doc_ptr || !loglik || !n_scored || D < 0 || n_foldin < 0)
        return fail(SABER_EINVAL, "saber_holdout_loglik: bad argument");
    if (m->parent) return fail(SABER_EINVAL, "saber_holdout_loglik: the model must be a context made by saber_init");
    if (doc_ptr[0] != 0) return fail(SABER_EINVAL, "saber_holdout_loglik: doc_ptr[0] must be 0");
    for (int64_t d = 0; d < D; d++)
        if (doc_ptr[d + 1] < doc_ptr[d]) return fail(SABER_EINVAL, "saber_holdout_loglik: doc_ptr decreases at document %lld", (long long)d);
    if (doc_ptr[D] > 0 && (!word_ids || !observed)) return fail(SABER_EINVAL, "saber_holdout_loglik: null token arrays");
    bool no_memory;
    int rc = holdout_loglik(m, doc_ptr, word_ids, observed, D, n_foldin, seed, z_init, z_out, loglik, n_scored, true, &no_memory);
    // where both layouts do not fit the host's memory: one after the other
    if (rc != SABER_OK && no_memory)
        rc = holdout_loglik(m, doc_ptr, word_ids, observed, D, n_foldin, seed, z_init, z_out, loglik, n_scored, false, &no_memory);
    return rc;
}

extern "C" int saber_get_z(saber_ctx *c, int32_t *z) {
    if (!c || !z) return fail(SABER_EINVAL, "saber_get_z: null argument");
    if (c->T == 0) return SABER_OK;
    try {
        if (c->n_slots) {   // document order is re-created chunk by chunk from the word-major copy
            // (the next chunk's token list comes in while this one's assignments go out, where there are two buffers: T = 20 M in four
            // chunks 4.4 -> 3.4 ms, with the documents, which nothing here reads, left out)
            std::vector<const Chunk *> list;
            for (const Chunk &ch : c->chunks) if (ch.ntok) list.push_back(&ch);
            const bool ahead = c->n_slots > 1;
            int s = -1, s_next = -1;
            for (size_t i = 0; i < list.size(); i++) {
                const Chunk &ch = *list[i];
                if (i == 0 || !ahead) SABER_TRY(stream_load(c, ch, false, &s)); else s = s_next;
                SABER_TRY(stream_wait(c, ch, s));
                if (c->z16)
                    hipLaunchKernelGGL((scatter_zwm_kernel<uint16_t>), dim3((unsigned)ch.ntiles), dim3(256), 0, c->stream,
                                       c->tiles + ch.tile0, c->slot_tok_t[s], (const uint16_t *)c->z_wm, (uint16_t *)c->slot_z[s]);
                else
                    hipLaunchKernelGGL((scatter_zwm_kernel<int32_t>), dim3((unsigned)ch.ntiles), dim3(256), 0, c->stream,
                                       c->tiles + ch.tile0, c->slot_tok_t[s], (const int32_t *)c->z_wm, (int32_t *)c->slot_z[s]);
                HIP_TRY(hipGetLastError());
                if (ahead && i + 1 < list.size()) SABER_TRY(stream_load(c, *list[i + 1], false, &s_next));
                SABER_TRY(pull_z(c, c->slot_z[s], ch.ntok, z + ch.t0));
                SABER_TRY(stream_release(c, s));
            }
            return SABER_OK;
        }
        return pull_z(c, c->z, c->T, z);
    } catch (const std::bad_alloc &) { return fail(SABER_ENOMEM, "saber_get_z: out of host memory"); }
}

extern "C" int saber_set_z(saber_ctx *c, const int32_t *z, uint32_t iter) {
    if (!c || (!z && c->T)) return fail(SABER_EINVAL, "saber_set_z: null argument");
    for (int64_t t = 0; t < c->T; t++)
        if (z[t] < 0 || z[t] >= c->K) return fail(SABER_EINVAL, "saber_set_z: topic %d at token %lld is outside [0,%d)", z[t], (long long)t, c->K);
    if (c->T && !c->n_slots) {
        int32_t *tmp = nullptr;
        SABER_TRY(dev_alloc(c->hooks, &tmp, (size_t)c->T));
        hipError_t e = hipMemcpy(tmp, z, sizeof(int32_t) * (size_t)c->T, hipMemcpyHostToDevice);
        if (e == hipSuccess) {
            if (c->z16)
                hipLaunchKernelGGL((z_from_i32_kernel<uint16_t>), dim3(grid_for(c->T, 256, 8192)), dim3(256), 0, c->stream, (uint16_t *)c->z, tmp, c->T);
            else
                hipLaunchKernelGGL((z_from_i32_kernel<int32_t>), dim3(grid_for(c->T, 256, 8192)), dim3(256), 0, c->stream, (int32_t *)c->z, tmp, c->T);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
        dev_free(c->hooks, tmp);
        if (e != hipSuccess) return fail(SABER_EDEVICE, "saber_set_z: %s", hipGetErrorString(e));
    }
    c->iter = iter;
    try { SABER_TRY(full_mstep(c, c->n_slots ? z : nullptr)); }
    catch (const std::bad_alloc &) { return fail(SABER_ENOMEM, "saber_set_z: out of host memory"); }
    return SABER_OK;
}

extern "C" int saber_get_iteration(saber_ctx *c, uint32_t *iter) {
    if (!c || !iter) return fail(SABER_EINVAL, "saber_get_iteration: null argument");
    *iter = c->iter;
    return SABER_OK;
}

// Device memory of one inspection call, cut from one block that the context keeps for the next call up to kWorkKept bytes (fresh
// device memory for every call took 0.9 of 1.8 ms: 100,000 tokens of 5 M, 400 rows of 1,500 topics).  It is memory of the context's
// device, whichever one the caller has current: later calls use it too.  A call that breaks off waits for what it has queued.
// Fresh memory of a few MB takes 0.3 ms whatever its size, below a MB 1 us: a block of more than a MB is a power of two of them, 8
// at least, so that a context's first calls share one.  The same two, a context's first 1.3 to 1.7 ms with memory for every
// call, 1.4 to 1.5 with a block of the size asked for, 0.8 to 1.2 so, later ones 0.91 to 1.9, 0.60 and 0.60; of 1,000 tokens of
// 100,000 and 400 rows of 100 topics 0.21, 0.19, 0.19, and 0.18, 0.16, 0.16.
constexpr size_t kWorkKept = (size_t)64 << 20;
struct WorkSpace {
    saber_ctx *c;
    char *base = nullptr;
    size_t at = 0;
    bool own = false, queued = false;
    explicit WorkSpace(saber_ctx *ctx) : c(ctx) {}
    ~WorkSpace() {
        if (queued) (void)hipStreamSynchronize(c->stream);
        if (own) dev_free(c->hooks, base);
    }
    static size_t rounded(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
    void drop() {
        dev_free(c->hooks, c->work);
        c->work = nullptr; c->work_bytes = 0;
    }
    int reserve(size_t bytes) {
        const DeviceScope scope(c->device);
        own = bytes > kWorkKept;
        if (own) {
            int rc = hook_alloc(c->hooks, (void **)&base, bytes);
            if (rc != SABER_OK && c->work) { drop(); rc = hook_alloc(c->hooks, (void **)&base, bytes); }
            return rc;
        }
        if (c->work_bytes < bytes) {
            drop();
            size_t block = (size_t)8 << 20;
            while (block < bytes) block *= 2;
            if (bytes <= ((size_t)1 << 20) || hook_alloc(c->hooks, &c->work, block) != SABER_OK) {   // (the larger one may not fit)
                block = bytes;
                SABER_TRY(hook_alloc(c->hooks, &c->work, block));
            }
            c->work_bytes = block;
        }
        base = (char *)c->work;
        return SABER_OK;
    }
    template <typename T> T *take(size_t n) { T *p = (T *)(base + at); at += rounded(n * sizeof(T)); return p; }
};

extern "C" int saber_token_probs(saber_ctx *c, const int64_t *tok, int64_t m, float *S, float *Q, float *p_sparse) {
    if (!c || (m > 0 && !tok) || m < 0) return fail(SABER_EINVAL, "saber_token_probs: bad argument");
    for (int64_t i = 0; i < m; i++)
        if (tok[i] < 0 || tok[i] >= c->T) return fail(SABER_EINVAL, "saber_token_probs: token index %lld is outside [0,%lld)", (long long)tok[i], (long long)c->T);
    if (m == 0) return SABER_OK;
    // S and Q of the tokens of a chunk (inspection mode of the sampling kernel), then the requested tokens of that
    // chunk are picked out and S / (S + Q) is formed, all on the device; the work space is sized for one chunk.
    // Fewer than an eighth of the tokens are marked, and only these worked on: 5 M tokens, K = 1,500, 100 of them 98 us, where a
    // pass over all took 221, 100,000 of them 0.25 ms, 600,000 1.04 and 1.07 (calls after a context's first).  Of more, S and Q of
    // all tokens are formed, runs of tokens sharing theirs; in chunks below 400,000 tokens as well, whose pass costs less than the
    // three launches that mark: T = 50,000, K = 68 66 us, 71 with marks; 200,000, K = 300 77 and 82; 500,000, K = 100 94 and 87.
    int64_t max_tok = 1;
    for (const Chunk &ch : c->chunks) max_tok = std::max(max_tok, ch.ntok);
    const bool few = m < c->T / 8 && max_tok >= 400'000;
    const size_t words = (size_t)(max_tok + 31) / 32, n = few ? (size_t)m : (size_t)max_tok;
    WorkSpace w(c);
    SABER_TRY(w.reserve(2 * w.rounded(n * sizeof(float)) + w.rounded(3 * (size_t)m * sizeof(float)) + w.rounded((size_t)m * sizeof(int64_t)) +
                        (few ? w.rounded((words + 1) * sizeof(uint2)) : 0)));
    float *dS = w.take<float>(n), *dQ = w.take<float>(n), *g3 = w.take<float>(3 * (size_t)m);
    int64_t *dtok = w.take<int64_t>((size_t)m);
    uint2 *marks = few ? w.take<uint2>(words + 1) : nullptr;   // (the last pair: the next number)
    HIP_TRY(hipMemcpy(dtok, tok, sizeof(int64_t) * (size_t)m, hipMemcpyHostToDevice));
    w.queued = true;
    // a thread per request: requests [i, i + n), as many as a grid takes, with f(i, n, grid)
    auto by_pieces = [&](auto f) -> int {
        for (int64_t i = 0, n; i < m; i += n) {
            n = std::min(m - i, 256 * most_blocks(256));
            f(i, n, dim3((unsigned)((n + 255) / 256)));
            HIP_TRY(hipGetLastError());
        }
        return SABER_OK;
    };
    for (const Chunk &ch : c->chunks) {
        if (ch.ntiles == 0) continue;
        int s = -1;
        if (c->n_slots) SABER_TRY(stream_acquire(c, ch, &s));
        if (few) {
            hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(2 * (int64_t)words + 2, 256, 8192)), dim3(256), 0, c->stream, (uint32_t *)marks, 0u, 2 * words + 2);
            HIP_TRY(hipGetLastError());
            SABER_TRY(by_pieces([&](int64_t i, int64_t n, dim3 grid) {
                hipLaunchKernelGGL(mark_tokens_kernel, grid, dim3(256), 0, c->stream, dtok + i, n, ch.t0, ch.ntok, marks);
            }));
            hipLaunchKernelGGL(number_tokens_kernel, dim3(grid_for((int64_t)words, 256)), dim3(256), 0, c->stream, marks, (int64_t)words, &marks[words].x);
            HIP_TRY(hipGetLastError());
        }
        EStepParams p = make_params(c, ch, s);
        p.marks = marks; p.out_S = dS; p.out_Q = dQ;
        SABER_TRY(launch_estep<MODE_PROBS>(c, c, ch, p));
        if (c->n_slots) SABER_TRY(stream_release(c, s));
        SABER_TRY(by_pieces([&](int64_t i, int64_t n, dim3 grid) {
            hipLaunchKernelGGL(gather_probs_kernel, grid, dim3(256), 0, c->stream, dS, dQ, marks, dtok + i, n, ch.t0, ch.ntok,
                               g3 + i, g3 + m + i, g3 + 2 * m + i);
        }));
    }
    HIP_TRY(hipStreamSynchronize(c->stream));
    w.queued = false;
    if (S) HIP_TRY(hipMemcpy(S, g3, sizeof(float) * (size_t)m, hipMemcpyDeviceToHost));
    if (Q) HIP_TRY(hipMemcpy(Q, g3 + m, sizeof(float) * (size_t)m, hipMemcpyDeviceToHost));
    if (p_sparse) HIP_TRY(hipMemcpy(p_sparse, g3 + 2 * m, sizeof(float) * (size_t)m, hipMemcpyDeviceToHost));
    return SABER_OK;
}

extern "C" int saber_get_phi(saber_ctx *c, const int32_t *words, int32_t m, float *phi, float *prefix) {
    if (!c || (m > 0 && !words) || m < 0) return fail(SABER_EINVAL, "saber_get_phi: bad argument");
    for (int32_t i = 0; i < m; i++)
        if (words[i] < 0 || words[i] >= c->V) return fail(SABER_EINVAL, "saber_get_phi: word %d is outside [0,%d)", words[i], c->V);
    if (m == 0) return SABER_OK;
    std::vector<int32_t> rows;
    try { rows.resize((size_t)m); } catch (const std::bad_alloc &) { return fail(SABER_ENOMEM, "saber_get_phi: out of host memory"); }
    for (int32_t i = 0; i < m; i++) rows[(size_t)i] = c->h_word_row[(size_t)words[i]];
    // assemble the requested Bhat rows on the device; the prefix rows are then rebuilt the way the dense branch does
    const size_t n = (size_t)m * (size_t)c->K;
    WorkSpace w(c);
    SABER_TRY(w.reserve((prefix ? 2 : 1) * w.rounded(n * sizeof(float)) + 2 * w.rounded((size_t)m * sizeof(int32_t))));
    float *drows = w.take<float>(n), *dout = prefix ? w.take<float>(n) : nullptr;
    int32_t *dw = w.take<int32_t>((size_t)m), *drow = w.take<int32_t>((size_t)m);
    HIP_TRY(hipMemcpy(dw, words, sizeof(int32_t) * (size_t)m, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(drow, rows.data(), sizeof(int32_t) * (size_t)m, hipMemcpyHostToDevice));
    w.queued = true;
    for (int64_t i = 0, k; i < m; i += k) {
        k = std::min<int64_t>(m - i, most_blocks(256));
        hipLaunchKernelGGL(phi_export_kernel, dim3((unsigned)k), dim3(256), 0, c->stream, drow + i, c->phi,
                           c->phi + (size_t)c->V_dense * (size_t)c->Kpad, c->wrec, c->lw_ent, c->lw_phi, c->K, c->Kpad, c->count_bits,
                           drows + (size_t)i * (size_t)c->K);
        HIP_TRY(hipGetLastError());
    }
    if (prefix) {
        const int64_t items = (int64_t)m * ((c->K + 63) / 64);
        hipLaunchKernelGGL(prefix_export_kernel, dim3((unsigned)items), dim3(64), 0, c->stream, drows, c->l3_64, dw, m,
                           c->K, c->n3, dout);
        HIP_TRY(hipGetLastError());
    }
    HIP_TRY(hipStreamSynchronize(c->stream));
    w.queued = false;
    if (phi) HIP_TRY(hipMemcpy(phi, drows, sizeof(float) * n, hipMemcpyDeviceToHost));
    if (prefix) HIP_TRY(hipMemcpy(prefix, dout, sizeof(float) * n, hipMemcpyDeviceToHost));
    return SABER_OK;
}

// ------------------------------------------------------------------------------------------------
// alias-table construction (measurement aid)
// ------------------------------------------------------------------------------------------------
extern "C" int saber_alias_build_probe(saber_ctx *c, const int32_t *words, int32_t m, float *prob, int32_t *alias,
                                       double *ms_build, int32_t *rows_built) {
    if (!c || m < 0 || (m > 0 && (!words || !prob || !alias)) || !ms_build)
        return fail(SABER_EINVAL, "saber_alias_build_probe: bad argument");
    if (c->parent) return fail(SABER_EINVAL, "saber_alias_build_probe: needs a context made by saber_init");
    std::vector<int32_t> rows;
    try { rows.resize((size_t)std::max(m, 1)); } catch (const std::bad_alloc &) { return fail(SABER_ENOMEM, "saber_alias_build_probe: out of host memory"); }
    for (int32_t i = 0; i < m; i++) {
        if (words[i] < 0 || words[i] >= c->V) return fail(SABER_EINVAL, "saber_alias_build_probe: word %d is outside [0,%d)", words[i], c->V);
        rows[(size_t)i] = c->h_word_row[(size_t)words[i]];
        if (rows[(size_t)i] < 0) return fail(SABER_EINVAL, "saber_alias_build_probe: word %d keeps a sparse row (no dense Bhat row to build from)", words[i]);
    }
    const int nrows = c->V_dense, K = c->K;
    if (rows_built) *rows_built = nrows;
    *ms_build = 0.0;
    if (nrows == 0) return m ? fail(SABER_EINVAL, "saber_alias_build_probe: no dense rows") : (int)SABER_OK;
    const size_t cells = (size_t)nrows * (size_t)K;
    if (cells * 20 > ((size_t)64 << 30)) return fail(SABER_ERANGE, "saber_alias_build_probe: tables of %zu bytes exceed 64 GB", cells * 20);
    double *scaled = nullptr; int32_t *stack = nullptr, *d_alias = nullptr, *d_rows = nullptr, *o_alias = nullptr;
    float *d_prob = nullptr, *o_prob = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto cleanup = [&]() {
        dev_free(c->hooks, scaled); dev_free(c->hooks, stack); dev_free(c->hooks, d_alias); dev_free(c->hooks, d_rows); dev_free(c->hooks, o_alias); dev_free(c->hooks, d_prob); dev_free(c->hooks, o_prob);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    };
    int rc;
    if ((rc = dev_alloc(c->hooks, &scaled, cells)) || (rc = dev_alloc(c->hooks, &stack, cells)) || (rc = dev_alloc(c->hooks, &d_alias, cells)) ||
        (rc = dev_alloc(c->hooks, &d_prob, cells)) || (rc = dev_alloc(c->hooks, &d_rows, (size_t)std::max(m, 1))) ||
        (rc = dev_alloc(c->hooks, &o_prob, (size_t)std::max(m, 1) * (size_t)K)) || (rc = dev_alloc(c->hooks, &o_alias, (size_t)std::max(m, 1) * (size_t)K))) {
        cleanup(); return rc;
    }
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) e = hipEventRecord(e0, c->stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(alias_build_kernel, dim3((unsigned)((nrows + 255) / 256)), dim3(256), 0, c->stream, c->phi, nrows, K,
                           c->Kpad, scaled, stack, d_prob, d_alias);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipEventRecord(e1, c->stream);
    if (e == hipSuccess && m) e = hipMemcpyAsync(d_rows, rows.data(), sizeof(int32_t) * (size_t)m, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess && m) {
        hipLaunchKernelGGL(alias_export_kernel, dim3(grid_for((int64_t)m * K, 256, 4096)), dim3(256), 0, c->stream, d_rows, m,
                           nrows, K, d_prob, d_alias, o_prob, o_alias);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e == hipSuccess && m) e = hipMemcpy(prob, o_prob, sizeof(float) * (size_t)m * (size_t)K, hipMemcpyDeviceToHost);
    if (e == hipSuccess && m) e = hipMemcpy(alias, o_alias, sizeof(int32_t) * (size_t)m * (size_t)K, hipMemcpyDeviceToHost);
    cleanup();
    if (e != hipSuccess) return fail(SABER_EDEVICE, "saber_alias_build_probe: %s", hipGetErrorString(e));
    *ms_build = (double)ms;
    return SABER_OK;
}

extern "C" int saber_get_alias(saber_ctx *c, const int32_t *words, int32_t m, float *prob, int32_t *alias) {
    if (!c || m < 0 || (m > 0 && (!words || !prob || !alias))) return fail(SABER_EINVAL, "saber_get_alias: bad argument");
    if (!c->alias_table) return fail(SABER_ESTATE, "saber_get_alias: the context keeps no alias tables (saber_options.ablation bit 2)");
    try {
        std::vector<uint2> rowbuf((size_t)c->K);
        for (int32_t i = 0; i < m; i++) {
            if (words[i] < 0 || words[i] >= c->V) return fail(SABER_EINVAL, "saber_get_alias: word %d is outside [0,%d)", words[i], c->V);
            const int32_t row = c->h_word_row[(size_t)words[i]];
            if (row < 0) return fail(SABER_ESTATE, "saber_get_alias: word %d keeps a sparse row", words[i]);
            HIP_TRY(hipMemcpy(rowbuf.data(), c->alias_table + (size_t)row * (size_t)c->K, sizeof(uint2) * (size_t)c->K, hipMemcpyDeviceToHost));
            for (int32_t k = 0; k < c->K; k++) {   // format conversion only
                memcpy(&prob[(size_t)i * (size_t)c->K + (size_t)k], &rowbuf[(size_t)k].x, sizeof(float));
                alias[(size_t)i * (size_t)c->K + (size_t)k] = (int32_t)rowbuf[(size_t)k].y;
            }
        }
    } catch (const std::bad_alloc &) { return fail(SABER_ENOMEM, "saber_get_alias: out of host memory"); }
    return SABER_OK;
}

extern "C" int saber_get_stats(saber_ctx *c, saber_stats *out) {
    if (!c || !out) return fail(SABER_EINVAL, "saber_get_stats: null argument");
    *out = c->stats;
    return SABER_OK;
}

extern "C" int saber_reset_stats(saber_ctx *c) {
    if (!c) return fail(SABER_EINVAL, "saber_reset_stats: null context");
    c->stats.iterations = 0; c->stats.ms_sample = c->stats.ms_count_dz = c->stats.ms_ck = c->stats.ms_phi = c->stats.ms_total = 0.0;
    c->stats.sample_launches = 0; c->stats.sum_tokens = c->stats.sum_tokens_dense = c->stats.sum_row_entries = c->stats.sum_row_fetch = c->stats.sum_light_entries = 0;
    return SABER_OK;
}

extern "C" int saber_get_stream(saber_ctx *c, void **s) {
    if (!c || !s) return fail(SABER_EINVAL, "saber_get_stream: null argument");
    *s = (void *)c->stream;
    return SABER_OK;
}

// ------------------------------------------------------------------------------------------------
// bandwidth probe (measurement aid; independent of any context)
// ------------------------------------------------------------------------------------------------
extern "C" int saber_bandwidth_probe(int64_t bytes, int32_t reps, double *gb_per_s) {
    if (bytes < 16 || reps < 1 || !gb_per_s) return fail(SABER_EINVAL, "saber_bandwidth_probe: bad argument");
    const size_t n16 = (size_t)bytes / 16;
    uint4 *src = nullptr, *dst = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = SABER_OK;
    auto cleanup = [&]() { dev_free(g_hooks, src); dev_free(g_hooks, dst); if (e0) (void)hipEventDestroy(e0); if (e1) (void)hipEventDestroy(e1); };
    if ((rc = dev_alloc(g_hooks, &src, n16)) || (rc = dev_alloc(g_hooks, &dst, n16))) { cleanup(); return rc; }
    hipError_t e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(fill_u32_kernel, dim3(8192), dim3(256), 0, 0, (uint32_t *)src, 1u, n16 * 4);
        hipLaunchKernelGGL(copy_probe_kernel, dim3(8192), dim3(256), 0, 0, src, dst, n16);   // warm-up
        e = hipEventRecord(e0, 0);
        for (int r = 0; r < reps; r++) hipLaunchKernelGGL(copy_probe_kernel, dim3(8192), dim3(256), 0, 0, src, dst, n16);
        if (e == hipSuccess) e = hipEventRecord(e1, 0);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipGetLastError();
    }
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    cleanup();
    if (e != hipSuccess) return fail(SABER_EDEVICE, "saber_bandwidth_probe: %s", hipGetErrorString(e));
    *gb_per_s = 2.0 * (double)(n16 * 16) * reps / ((double)ms * 1e-3) / 1e9;   // read + write
    return SABER_OK;
}
