// C-ABI entry points of libsvdp (see include/svdp.h): host-side validation,
// workspace carving and kernel launches.  No allocation, no synchronisation,
// no state kept between calls (everything follows from a call's arguments).
#include "../../include/svdp.h"

#include <hip/hip_runtime.h>

#include "svdp_kernels.h"
#include "svdp_rows_mfma.h"
#include "svdp_predict_small.h"
#include "svdp_rows_seq.h"
#include "svdp_calib.h"
#include "svdp_calib_stats.h"
#include "svdp_whiten.h"
#include "svdp_eigtop.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <functional>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

namespace {

using namespace svdp;

constexpr int XP_MAX_BLOCKS = 128;    // stage-1 row slabs of P (d <= 16384)
constexpr size_t ALIGN = 256;
constexpr size_t LDS_DEFAULT = 64 * 1024;     // dynamic LDS a kernel may use without asking
constexpr int MAX_DEVICES = 64;

inline size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }
inline int nb_of(int B) { return B <= 1 ? 1 : B <= 2 ? 2 : B <= 4 ? 4 : 8; }
inline int vec_of(int dt) { return dt == SVDP_F32 ? 4 : 8; }
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
inline bool bad_batch(int B) { return B < 1 || B > SVDP_MAX_BATCH; }

constexpr uint32_t ALL_FLAGS =
    SVDP_FLAG_DRELU | SVDP_FLAG_REVALIDATE | SVDP_FLAG_ENGINE_VECTOR | SVDP_FLAG_ENGINE_MATRIX;

svdp_status check_shape(int d, int D, int r, int dt)
{
    if (dt != SVDP_F32 && dt != SVDP_BF16) return SVDP_ERR_UNSUPPORTED;
    if (d <= 0 || D <= 0 || r <= 0) return SVDP_ERR_INVALID_ARG;
    const int e = vec_of(dt);
    if (D % 64 != 0 || d % e != 0 || r % e != 0) return SVDP_ERR_UNSUPPORTED;
    if (r > 2048 || d > 16384) return SVDP_ERR_UNSUPPORTED;
    return SVDP_OK;
}

svdp_status check_layer(const svdp_layer *L, bool need_pred, bool need_ffn)
{
    if (L == nullptr) return SVDP_ERR_INVALID_ARG;
    const svdp_status st = check_shape(L->d, L->D, L->r, L->wdtype);
    if (st != SVDP_OK) return st;
    if (need_pred && (!L->P || !L->Q || !L->b || !aligned16(L->P) || !aligned16(L->Q) ||
                      (reinterpret_cast<uintptr_t>(L->b) & 3u)))
        return SVDP_ERR_INVALID_ARG;
    if (need_ffn && (!L->W_gate || !L->W_up || !L->W_downT || !aligned16(L->W_gate) ||
                     !aligned16(L->W_up) || !aligned16(L->W_downT)))
        return SVDP_ERR_INVALID_ARG;
    if (L->flags & ~ALL_FLAGS) return SVDP_ERR_INVALID_ARG;
    if ((L->flags & SVDP_FLAG_ENGINE_VECTOR) && (L->flags & SVDP_FLAG_ENGINE_MATRIX)) return SVDP_ERR_INVALID_ARG;
    return SVDP_OK;
}

// Workspace layout (all offsets 256-byte aligned):
//   tpart [XP_MAX_BLOCKS + 1][NB][r] f32 | mask [D/64] u64 | nnz i32 | ypart [ROWS_BLOCKS][NB][d] f32
struct Workspace {
    float *tpart;
    uint64_t *mask;
    int32_t *nnz;
    float *ypart;
    size_t bytes;
};

Workspace carve(void *base, int d, int D, int r, int NB)
{
    Workspace w;
    char *p = static_cast<char *>(base);
    size_t off = 0;
    w.tpart = reinterpret_cast<float *>(p + off);
    off += align_up((size_t)(XP_MAX_BLOCKS + 1) * NB * r * 4);     // partials, then the finished t
    w.mask = reinterpret_cast<uint64_t *>(p + off);
    off += align_up((size_t)D / 64 * 8);
    w.nnz = reinterpret_cast<int32_t *>(p + off);
    off += ALIGN;
    w.ypart = reinterpret_cast<float *>(p + off);
    off += align_up((size_t)ROWS_BLOCKS * NB * d * 4);
    w.bytes = off;
    return w;
}

// Enqueues a kernel.  Straight to hipLaunchKernel: the <<<>>> form goes through a push and a pop of the launch
// configuration besides (2.4 -> 2.25 us a launch of twenty arguments), and launches are what bounds small calls: a list of two
// rows 9.7 -> 8.5 us, the step of d = 256, D = 1024 12.7 -> 11.6 (10.5 to 12.5 by the host it runs on).  A refused launch is the
// last error, which hip_status() reports.
template <typename... P, typename... A>
inline void launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t st, A &&...args)
{
    [&](P... p) {
        void *at[] = {const_cast<void *>(static_cast<const void *>(&p))...};
        (void)hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, at, lds, st);
    }(std::forward<A>(args)...);
}

inline svdp_status hip_status(hipError_t e)
{
    if (e == hipSuccess) e = hipGetLastError();
    else (void)hipGetLastError();
    return e == hipSuccess ? SVDP_OK : SVDP_ERR_HIP;
}

// Dynamic LDS above the default limit has to be enabled per kernel and device once.  What was
// enabled is remembered per kernel (the template parameter is the kernel itself) and device;
// the driver call is made under a lock, so that the remembered size never runs ahead of it.
std::mutex g_grant_mutex;
template <auto Kernel>
bool grant_lds(size_t bytes)
{
    static std::atomic<int> granted[MAX_DEVICES];
    if (bytes <= LDS_DEFAULT) return true;
    if (bytes > LDS_MAX) return false;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        (void)hipGetLastError();
        return false;
    }
    if ((int)bytes <= granted[dev].load(std::memory_order_acquire)) return true;
    std::lock_guard<std::mutex> lock(g_grant_mutex);
    if ((int)bytes <= granted[dev].load(std::memory_order_relaxed)) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    granted[dev].store((int)bytes, std::memory_order_release);
    return true;
}

// ---- which kernels a call uses and how much LDS they need: pure host arithmetic ----

enum Engine { ENGINE_AUTO = 0, ENGINE_VECTOR = 1, ENGINE_MATRIX = 2 };
inline Engine engine_of(const svdp_layer *L)
{
    return (L->flags & SVDP_FLAG_ENGINE_VECTOR) ? ENGINE_VECTOR
                                                : (L->flags & SVDP_FLAG_ENGINE_MATRIX) ? ENGINE_MATRIX : ENGINE_AUTO;
}

inline int xp_slabs(int d) { return (d + XP_ROWS - 1) / XP_ROWS; }        // partials of t; <= XP_MAX_BLOCKS since d <= 16384

template <typename W, int NB>
size_t xp_lds(const svdp_layer *)
{
    constexpr int VEC = Elem<W>::VEC;
    const size_t outs = (size_t)NB * XP_COLS;
    const size_t parts = XP_THREADS / outs >= 1 ? XP_THREADS / outs : 1;
    const size_t nsub = XP_THREADS / (XP_COLS / VEC);
    return ((size_t)NB * XP_ROWS + nsub * (outs + 1) + parts * outs) * 4;
}

// Whether the scores run on the matrix cores: from three tokens on unless the caller wants the vector units; for fewer where
// the caller wants it and the layer is a plain one (bf16, whole column blocks held in registers).
template <typename W, int NB>
bool scores_on_matrix(const svdp_layer *L)
{
    const Engine engine = engine_of(L);
    if (NB >= 4) return engine != ENGINE_VECTOR;
    return engine == ENGINE_MATRIX && std::is_same<W, bf16>::value && L->r % 32 == 0 && L->r <= 512;
}
template <int NB>
constexpr int scores_threads() { return NB <= 2 ? 512 : 256; }
template <typename W, int NB>
size_t scores_lds(const svdp_layer *L)
{
    if (scores_on_matrix<W, NB>(L)) return scm_lds<W>(NB, L->r);
    const size_t thr = scores_threads<NB>();
    const size_t tsp = (size_t)NB * L->r > thr * 4 ? (size_t)NB * L->r : thr * 4;
    return ((size_t)NB * L->r + (size_t)NB * SC_SLAB + tsp) * 4;
}

enum RowsKind { ROWS_VECTOR = 0, ROWS_SEQ = 1, ROWS_MATRIX = 2 };
struct RowsPlan {
    RowsKind kind;
    int max_chunk;      // LDS row capacity of a block
    int min_chunk;      // fewest rows a block takes (short lists use fewer blocks)
    size_t lds;
    bool split;         // gate/up kernel, then the down projection over column slices (k_down_slices)
};

// Split organisation: where its buffers lie inside the workspace's partial-y region [ROWS_BLOCKS][NB][d]: the DOWN_RG partial
// y's, then h [D][NB], then the list [D].
inline size_t split_h_offset(int d, int NB) { return align_up((size_t)DOWN_RG * NB * d * 4); }
inline size_t split_list_offset(int d, int D, int NB) { return split_h_offset(d, NB) + align_up((size_t)D * NB * 4); }
inline bool split_fits(int d, int D, int NB)
{
    return (D + DOWN_RG - 1) / DOWN_RG <= DS_MAX_CHUNK &&
           split_list_offset(d, D, NB) + (size_t)D * 4 <= (size_t)ROWS_BLOCKS * NB * d * 4;
}

// d * D from which the matrix engine's two row kernels are chosen over a list, and above which over all rows, if each block of
// the vector kernel has more than three
constexpr size_t ROWS_MATRIX_MIN = 2 << 20, ROWS_MATRIX_DENSE_MIN = 1 << 20;
constexpr int ROWS_MATRIX_DENSE_ROWS = 3 * ROWS_BLOCKS;
template <typename W, int NB, int MODE = ROWS_MASK>
RowsPlan plan_rows(const svdp_layer *L)
{
    const int d = L->d, D = L->D;
    RowsPlan p;
    p.split = false;
    if ((L->flags & SVDP_FLAG_REVALIDATE) != 0) {
        p.kind = ROWS_SEQ;
        p.min_chunk = ROWS_MIN_CHUNK;
        p.max_chunk = rows_max_chunk(D, p.min_chunk, ROWS_UB);
        p.lds = (size_t)NB * d * sizeof(W) + ((size_t)2 * NB * p.max_chunk + (size_t)3 * p.max_chunk) * 4;
        return p;
    }
    if (std::is_same<W, bf16>::value) {
        const Engine engine = engine_of(L);
        // Rows alone, vector -> matrix, at 30 / 60 % of the rows, eight tokens (us): d x D = 512 x 2560 11.4 -> 12.2 / 13.2 ->
        // 12.6, 768 x 3072 13.4 -> 12.6 / 14.3 -> 13.1, 1024 x 4672 15.8 -> 13.8 / 19.5 -> 15.5, 2432 x 12864 30.1 -> 24.3 /
        // 43.0 -> 35.6; below 2 M elements the launch more is not earned back.  Rows that end inside a 128-byte line, whole
        // step: d x D = 3128 x 12160, B = 8 78.6 -> 67.8, 2104 x 8064, B = 6 37.5 -> 30.9.
        // Four tokens, whole step with the sum of the partial outputs, scores on the matrix cores either way, list of 0.33 to 0.4 /
        // 0.55 to 0.6 of the rows, weights from memory: vector ahead or level.  512 x 2560 16.5 -> 18.8 / 17.8 -> 19.5,
        // 1024 x 4672 20.6 -> 22.4 / 23.4 -> 24.9, 2432 x 12864 38.4 -> 38.8 / 46.9 -> 46.3, 3584 x 18944 57.2 -> 60.1 / 76.2 ->
        // 77.2, 4096 x 11008 41.5 -> 42.4 / 53.1 -> 54.7; from the cache the same within 1 us.
        // Over all rows, eight (five) tokens: 256 x 5120 17.9 -> 14.8 (18.0 -> 14.8), 512 x 4032 16.4 -> 13.7 (15.7 -> 13.7),
        // 1000 x 1088 16.1 -> 12.3 (14.3 -> 12.2), 1024 x 1984 15.0 -> 13.1 (13.4 -> 13.0), 2048 x 960 17.6 -> 15.4 (15.0 -> 15.1);
        // below: 1024 x 1024 13.7 -> 12.6 (12.0 -> 12.6), 512 x 1024 11.1 -> 11.7, 2048 x 640 14.8 -> 15.2 (12.9 -> 14.9), 3072 x 384 16.2 -> 18.4 (14.3 -> 18.0).
        const size_t size = (size_t)d * D;
        const bool large = size >= ROWS_MATRIX_MIN ||
                           (MODE == ROWS_DENSE && size > ROWS_MATRIX_DENSE_MIN && D > ROWS_MATRIX_DENSE_ROWS);
        const bool want = engine == ENGINE_MATRIX || (engine == ENGINE_AUTO && NB >= 8 && large);
        if (want) {
            p.kind = ROWS_MATRIX;
            p.min_chunk = MF_ROWS;
            p.max_chunk = rows_max_chunk(D, MF_ROWS, MF_ROWS);
            p.lds = mf_lds(d, D, NB);
            p.split = true;
            if (p.lds <= LDS_MAX && split_fits(d, D, NB)) return p;
            p.split = false;
        }
    }
    p.kind = ROWS_VECTOR;
    p.min_chunk = ROWS_MIN_CHUNK;
    p.max_chunk = rows_max_chunk(D, p.min_chunk, ROWS_UB);
    p.lds = (size_t)NB * d * sizeof(W) + ((size_t)NB * p.max_chunk + p.max_chunk) * 4;
    return p;
}

// dispatch on (dtype, batch capacity): f(W tag, NB constant)
template <typename T>
struct Tag {
    using type = T;
};
template <typename F>
auto dispatch(int dt, int NBv, F &&f)
{
    auto on_nb = [&](auto wtag) {
        switch (NBv) {
        case 1: return f(wtag, std::integral_constant<int, 1>{});
        case 2: return f(wtag, std::integral_constant<int, 2>{});
        case 4: return f(wtag, std::integral_constant<int, 4>{});
        default: return f(wtag, std::integral_constant<int, 8>{});
        }
    };
    return dt == SVDP_F32 ? on_nb(Tag<float>{}) : on_nb(Tag<bf16>{});
}

// Everything every kernel of the layer needs fits the LDS of a compute unit (pure).
bool layer_fits(const svdp_layer *L, int NBv)
{
    return dispatch(L->wdtype, NBv, [&](auto wt, auto nb) {
        using W = typename decltype(wt)::type;
        constexpr int NB = decltype(nb)::value;
        return xp_lds<W, NB>(L) <= LDS_MAX && scores_lds<W, NB>(L) <= LDS_MAX && plan_rows<W, NB>(L).lds <= LDS_MAX;
    });
}

svdp_status check_ws(const svdp_layer *L, int B, void *ws, size_t ws_bytes, Workspace *out)
{
    if (!layer_fits(L, nb_of(B))) return SVDP_ERR_UNSUPPORTED;
    if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & (ALIGN - 1))) return SVDP_ERR_WORKSPACE;
    *out = carve(ws, L->d, L->D, L->r, nb_of(B));
    if (ws_bytes < out->bytes) return SVDP_ERR_WORKSPACE;
    return SVDP_OK;
}

// ---- preparation (LDS grants; nothing is enqueued) and launch, per kernel ----

// The stacked benchmark's glue folded into the first kernel of a step (svdp_ffn_step_glued).
struct GlueArgs {
    const float *y_prev;
    const float *shift;
    float eps;
    void *x_out;
};

template <typename W, int NB>
bool prepare_xP(const svdp_layer *L, bool glue)
{
    const size_t lds = xp_lds<W, NB>(L);
    return glue ? grant_lds<k_xP<W, NB, true>>(lds) : grant_lds<k_xP<W, NB, false>>(lds);
}

template <typename W, int NB>
svdp_status launch_xP(const svdp_layer *L, const void *x, int B, float *tpart, int *nt_out, hipStream_t st,
                      const GlueArgs *glue)
{
    const int d = L->d, r = L->r;
    const int nt = xp_slabs(d);
    const int ncs = (r + XP_COLS - 1) / XP_COLS;
    const size_t lds = xp_lds<W, NB>(L);
    if (glue != nullptr) {
        launch((k_xP<W, NB, true>), dim3(nt, ncs), dim3(XP_THREADS), lds, st, static_cast<const W *>(L->P),
               static_cast<const W *>(x), B, d, r, tpart, glue->y_prev, glue->shift, glue->eps,
               static_cast<W *>(glue->x_out));
    } else {
        launch((k_xP<W, NB, false>), dim3(nt, ncs), dim3(XP_THREADS), lds, st,
               static_cast<const W *>(L->P), static_cast<const W *>(x), B, d, r, tpart, nullptr, nullptr,
               0.f, nullptr);
    }
    *nt_out = nt;
    return hip_status(hipSuccess);
}

// lanes per row of the vector score kernel: 2^k >= 16-byte column groups per row of Q, 8..64
template <typename W>
int scores_lpr_log2(const svdp_layer *L)
{
    const int cg = L->r / Elem<W>::VEC;
    return cg <= 8 ? 3 : cg <= 16 ? 4 : cg <= 32 ? 5 : 6;
}

template <typename W, int NB, typename F>
auto with_scores_kernel(const svdp_layer *L, F &&f)
{
    constexpr int THR = scores_threads<NB>();
    switch (scores_lpr_log2<W>(L)) {
    case 3: return f(std::integral_constant<decltype(&k_scores<W, NB, 3, THR>), &k_scores<W, NB, 3, THR>>{});
    case 4: return f(std::integral_constant<decltype(&k_scores<W, NB, 4, THR>), &k_scores<W, NB, 4, THR>>{});
    case 5: return f(std::integral_constant<decltype(&k_scores<W, NB, 5, THR>), &k_scores<W, NB, 5, THR>>{});
    default: return f(std::integral_constant<decltype(&k_scores<W, NB, 6, THR>), &k_scores<W, NB, 6, THR>>{});
    }
}

// The matrix score kernel for a layer: column blocks of Q that a wave holds and partials of t that a thread requests together, both
// nearly as many as there are, since a request for what is not there is not free.
template <typename W, int NB, typename F>
auto with_matrix_scores_kernel(const svdp_layer *L, F &&f)
{
    const int nkb = (L->r + scm_block<W>() - 1) / scm_block<W>(), nt = xp_slabs(L->d);
    auto of = [&](auto kb, auto parts) {
        constexpr auto k = &k_scores_mfma<W, NB, decltype(kb)::value, decltype(parts)::value>;
        return f(std::integral_constant<decltype(k), k>{});
    };
    auto with_parts = [&](auto kb) {
        if constexpr (NB >= 4) {               // one and two tokens come here only on the caller's wish
            if (nt <= SCM_NT / 4) return of(kb, std::integral_constant<int, SCM_NT / 4>{});
            if ((nt - 1) % SCM_NT < SCM_NT / 2) return of(kb, std::integral_constant<int, SCM_NT / 2>{});
        }
        return of(kb, std::integral_constant<int, SCM_NT>{});
    };
    if (nkb <= SCM_KB / 4) return with_parts(std::integral_constant<int, SCM_KB / 4>{});
    if (nkb <= SCM_KB / 2) return with_parts(std::integral_constant<int, SCM_KB / 2>{});
    if (nkb <= SCM_KB * 3 / 4) return with_parts(std::integral_constant<int, SCM_KB * 3 / 4>{});
    return with_parts(std::integral_constant<int, SCM_KB>{});
}

template <typename W, int NB>
bool prepare_scores(const svdp_layer *L)
{
    const size_t lds = scores_lds<W, NB>(L);
    if (scores_on_matrix<W, NB>(L)) return with_matrix_scores_kernel<W, NB>(L, [&](auto k) { return grant_lds<decltype(k)::value>(lds); });
    return with_scores_kernel<W, NB>(L, [&](auto k) { return grant_lds<decltype(k)::value>(lds); });
}

template <typename W, int NB>
svdp_status launch_scores(const svdp_layer *L, const float *tpart, int nt, int B, float *s_out, uint64_t *mask_out,
                          hipStream_t st)
{
    const size_t lds = scores_lds<W, NB>(L);
    if (scores_on_matrix<W, NB>(L)) {
        with_matrix_scores_kernel<W, NB>(L, [&](auto k) {
            launch(decltype(k)::value, dim3(L->D / SC_SLAB), dim3(SCM_THREADS), lds, st, static_cast<const W *>(L->Q), L->b,
                   tpart, nt, L->r, B, mask_out, s_out, L->D);
            return 0;
        });
        return hip_status(hipSuccess);
    }
    // block size: 512 threads for one or two tokens (short critical path), 256 for larger batches
    // (fewer wavefronts repeating the per-wave overhead); measured on the 7B and Mistral shapes
    // threads per float4 column of t: no more than there are partials to add
    const int npg = std::max(1, std::min(scores_threads<NB>() / (NB * L->r / 4), nt));
    with_scores_kernel<W, NB>(L, [&](auto k) {
        launch(decltype(k)::value, dim3(L->D / SC_SLAB), dim3(scores_threads<NB>()), lds, st,
               static_cast<const W *>(L->Q), L->b, tpart, nt, npg, L->r, B, mask_out, s_out, L->D);
        return 0;
    });
    return hip_status(hipSuccess);
}

template <typename W, int NB, int MODE>
bool prepare_rows(const svdp_layer *L)
{
    const RowsPlan p = plan_rows<W, NB, MODE>(L);
    if (p.kind == ROWS_SEQ) return grant_lds<k_rows_seq<W, NB, MODE>>(p.lds);
    if constexpr (std::is_same<W, bf16>::value) {
        if (p.kind == ROWS_MATRIX) return grant_lds<k_gate_up_mfma<NB, MODE>>(p.lds);
    }
    return grant_lds<k_rows<W, NB, MODE>>(p.lds);
}

// Gate, up and down over the list.  With y == nullptr the final sum of the partial results is left out (they
// stay in the workspace): the row work by itself, for timing.
template <typename W, int NB, int MODE>
svdp_status launch_rows(const svdp_layer *L, const void *x, int B, const uint64_t *mask, const int32_t *idx_in,
                        const int32_t *nnz_in, int32_t *idx_out, int32_t *nnz_out, const Workspace &w, float *y,
                        hipStream_t st)
{
    const RowsPlan p = plan_rows<W, NB, MODE>(L);
    const int d = L->d, D = L->D;
    const W *Wg = static_cast<const W *>(L->W_gate), *Wu = static_cast<const W *>(L->W_up);
    const W *Wd = static_cast<const W *>(L->W_downT), *xs = static_cast<const W *>(x);
    const void *list = MODE == ROWS_MASK ? static_cast<const void *>(mask) : idx_in;
    const int dB = d | B << 16;                 // d <= 16384: the kernels' arguments that come in registers are few
    bool matrix = false;
    if constexpr (std::is_same<W, bf16>::value) {
        matrix = p.kind == ROWS_MATRIX;
        if (matrix) {
            // gate/up kernel, then the down projection over column slices, which leaves DOWN_RG partial outputs
            char *region = reinterpret_cast<char *>(w.ypart);
            float *hbuf = reinterpret_cast<float *>(region + split_h_offset(d, NB));
            int32_t *lst = reinterpret_cast<int32_t *>(region + split_list_offset(d, D, NB));
            launch((k_gate_up_mfma<NB, MODE>), dim3(ROWS_BLOCKS), dim3(ROWS_THREADS), p.lds, st, xs, list, Wg, Wu, nnz_in, dB,
                   D, L->flags, idx_out, nnz_out, w.nnz, hbuf, lst);
            launch((k_down_slices<NB, MODE == ROWS_DENSE>), dim3((d + DS_SW - 1) / DS_SW, DOWN_RG), dim3(DS_THREADS), 0, st,
                   Wd, lst, MODE == ROWS_DENSE ? nullptr : w.nnz, D, d, hbuf, w.ypart);
        }
    }
    if (matrix) {
        // launched above
    } else if (p.kind == ROWS_SEQ) {
        launch((k_rows_seq<W, NB, MODE>), dim3(ROWS_BLOCKS), dim3(ROWS_THREADS), p.lds, st, xs, list, Wg, Wu, Wd, nnz_in, dB, D,
               L->flags, idx_out, nnz_out, w.nnz, w.ypart);
    } else {
        launch((k_rows<W, NB, MODE>), dim3(ROWS_BLOCKS), dim3(ROWS_THREADS), p.lds, st, xs, list, Wg, Wu, Wd, nnz_in, dB, D,
               L->flags, idx_out, nnz_out, w.nnz, w.ypart);
    }
    if (y != nullptr) {
        // all rows: the number of partial outputs is known here
        const int min_chunk = p.split ? DOWN_MIN_CHUNK : p.min_chunk, G = p.split ? DOWN_RG : ROWS_BLOCKS;
        const int chunk = std::max(min_chunk, (D + G - 1) / G), parts = (D + chunk - 1) / chunk;
        launch(k_reduce_y, dim3((d / 4 + RED_COLS - 1) / RED_COLS, B), dim3(RED_COLS * RED_SEGS), 0, st, w.ypart,
               MODE == ROWS_DENSE ? nullptr : w.nnz, y, parts, NB, d);
    }
    return hip_status(hipSuccess);
}

template <typename W, int NB>
bool tsum_needed(const svdp_layer *L)
{
    // finish t once instead of in every score block (the vector score kernel splits the partial
    // list over threads through LDS, which costs more than a launch from 4 tokens up)
    return NB >= 4 && L->d > XP_ROWS && !scores_on_matrix<W, NB>(L);
}

// One token and a P of at most PS_TILES tiles: both predictor stages in one launch (k_predict_small).
template <typename W>
bool predict_small(const svdp_layer *L)
{
    const int tiles = xp_slabs(L->d) * ((L->r + XP_COLS - 1) / XP_COLS);
    return tiles <= PS_TILES && !scores_on_matrix<W, 1>(L);
}

template <typename W>
svdp_status launch_predict_small(const svdp_layer *L, const void *x, float *s, uint64_t *mask, hipStream_t st)
{
    auto go = [&](auto lpr) {
        launch((k_predict_small<W, decltype(lpr)::value>), dim3(L->D / SC_SLAB), dim3(PS_THREADS),
               ps_lds<W>(L->d, L->r), st, static_cast<const W *>(L->P), static_cast<const W *>(L->Q), L->b,
               static_cast<const W *>(x), L->d, L->r, s, mask);
        return hip_status(hipSuccess);
    };
    switch (scores_lpr_log2<W>(L)) {                  // r <= 32 PS_TILES: at most 32 column groups
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
    default: return go(std::integral_constant<int, 5>{});
    }
}

template <typename W, int NB>
svdp_status run_predict(const svdp_layer *L, const void *x, int B, float *s, uint64_t *mask, const Workspace &w,
                        hipStream_t st, const GlueArgs *glue)
{
    if (NB == 1 && glue == nullptr && predict_small<W>(L)) return launch_predict_small<W>(L, x, s, mask, st);
    int nt = 0;
    svdp_status e = launch_xP<W, NB>(L, x, B, w.tpart, &nt, st, glue);
    if (e != SVDP_OK) return e;
    if (tsum_needed<W, NB>(L)) {
        const int count = NB * L->r;
        float *t = w.tpart + (size_t)XP_MAX_BLOCKS * NB * L->r;
        launch(k_tsum, dim3((count + 255) / 256), dim3(256), 0, st, w.tpart, nt, count, t);
        e = hip_status(hipSuccess);
        if (e != SVDP_OK) return e;
        return launch_scores<W, NB>(L, t, 1, B, s, mask, st);
    }
    return launch_scores<W, NB>(L, w.tpart, nt, B, s, mask, st);
}

// The whole step: every LDS grant first (on failure nothing has been enqueued), then the launches.
svdp_status step_impl(const svdp_layer *L, const void *x, int B, float *y, uint64_t *mask_out, int32_t *idx_out,
                      int32_t *nnz_out, const Workspace &w, hipStream_t st, const GlueArgs *glue)
{
    return dispatch(L->wdtype, nb_of(B), [&](auto wt, auto nb) -> svdp_status {
        using W = typename decltype(wt)::type;
        constexpr int NB = decltype(nb)::value;
        if (!prepare_xP<W, NB>(L, glue != nullptr) || !prepare_scores<W, NB>(L) || !prepare_rows<W, NB, ROWS_MASK>(L))
            return SVDP_ERR_UNSUPPORTED;
        uint64_t *mask = mask_out ? mask_out : w.mask;
        const svdp_status e = run_predict<W, NB>(L, x, B, nullptr, mask, w, st, glue);
        if (e != SVDP_OK) return e;
        // with the glue, x is made by the first kernel (from x_prev = x) and the row kernel reads it from x_out
        const void *xr = glue != nullptr ? glue->x_out : x;
        return launch_rows<W, NB, ROWS_MASK>(L, xr, B, mask, nullptr, nullptr, idx_out, nnz_out, w, y, st);
    });
}

// ---- the scratch buffer of svdp_ffn_step_static: one array per device, in the library's image ----
__device__ __align__(256) unsigned char g_static_scratch[SVDP_STATIC_SCRATCH_BYTES];

std::mutex g_scratch_mutex;
std::atomic<void *> g_scratch_ptr[MAX_DEVICES];

// Address of the current device's copy of the array (looked up once per device).
void *static_scratch()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        (void)hipGetLastError();
        return nullptr;
    }
    void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p != nullptr) return p;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (p != nullptr) return p;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)) != hipSuccess || p == nullptr) {
        (void)hipGetLastError();
        return nullptr;
    }
    g_scratch_ptr[dev].store(p, std::memory_order_release);
    return p;
}

#include "svdp_whiten_run.h"
#include "svdp_eigtop_run.h"
#include "svdp_whiten_call.h"

}  // namespace

extern "C" {

size_t svdp_workspace_bytes(const svdp_layer *layer, int32_t max_batch)
{
    if (layer == nullptr || bad_batch(max_batch)) return 0;
    if (check_shape(layer->d, layer->D, layer->r, layer->wdtype) != SVDP_OK) return 0;
    if ((layer->flags & ~ALL_FLAGS) ||
        ((layer->flags & SVDP_FLAG_ENGINE_VECTOR) && (layer->flags & SVDP_FLAG_ENGINE_MATRIX)))
        return 0;
    if (!layer_fits(layer, nb_of(max_batch))) return 0;
    return carve(nullptr, layer->d, layer->D, layer->r, nb_of(max_batch)).bytes;
}

svdp_status svdp_predict(const svdp_layer *layer, const void *x, int32_t B, float *s, void *ws, size_t ws_bytes,
                         void *stream)
{
    svdp_status st = check_layer(layer, true, false);
    if (st != SVDP_OK) return st;
    if (x == nullptr || s == nullptr || bad_batch(B) || !aligned16(x)) return SVDP_ERR_INVALID_ARG;
    Workspace w;
    st = check_ws(layer, B, ws, ws_bytes, &w);
    if (st != SVDP_OK) return st;
    return dispatch(layer->wdtype, nb_of(B), [&](auto wt, auto nb) -> svdp_status {
        using W = typename decltype(wt)::type;
        constexpr int NB = decltype(nb)::value;
        if (!prepare_xP<W, NB>(layer, false) || !prepare_scores<W, NB>(layer)) return SVDP_ERR_UNSUPPORTED;
        return run_predict<W, NB>(layer, x, B, s, nullptr, w, static_cast<hipStream_t>(stream), nullptr);
    });
}

svdp_status svdp_compact(const float *s, int32_t B, int32_t D, uint64_t *mask, int32_t *idx, int32_t *nnz,
                         void *ws, size_t ws_bytes, void *stream)
{
    (void)ws;
    (void)ws_bytes;
    if (s == nullptr || mask == nullptr || idx == nullptr || nnz == nullptr || bad_batch(B) || D <= 0) return SVDP_ERR_INVALID_ARG;
    if (D % 64 != 0) return SVDP_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    launch(k_mask_from_scores, dim3((D / 64 + 3) / 4), dim3(256), 0, st, s, B, D, mask);
    const svdp_status e = hip_status(hipSuccess);
    if (e != SVDP_OK) return e;
    launch(k_compact_scan, dim3(1), dim3(SCAN_THREADS), 0, st, mask, D / 64, idx, nnz);
    return hip_status(hipSuccess);
}

svdp_status svdp_sparse_ffn(const svdp_layer *layer, const void *x, int32_t B, const int32_t *idx,
                            const int32_t *nnz, float *y, void *ws, size_t ws_bytes, void *stream)
{
    svdp_status st = check_layer(layer, false, true);
    if (st != SVDP_OK) return st;
    if (x == nullptr || y == nullptr || idx == nullptr || nnz == nullptr || bad_batch(B) || !aligned16(x) ||
        !aligned16(y))
        return SVDP_ERR_INVALID_ARG;
    Workspace w;
    st = check_ws(layer, B, ws, ws_bytes, &w);
    if (st != SVDP_OK) return st;
    return dispatch(layer->wdtype, nb_of(B), [&](auto wt, auto nb) -> svdp_status {
        using W = typename decltype(wt)::type;
        constexpr int NB = decltype(nb)::value;
        if (!prepare_rows<W, NB, ROWS_LIST>(layer)) return SVDP_ERR_UNSUPPORTED;
        return launch_rows<W, NB, ROWS_LIST>(layer, x, B, nullptr, idx, nnz, nullptr, nullptr, w, y,
                                             static_cast<hipStream_t>(stream));
    });
}

svdp_status svdp_dense_ffn(const svdp_layer *layer, const void *x, int32_t B, float *y, void *ws, size_t ws_bytes,
                           void *stream)
{
    svdp_status st = check_layer(layer, false, true);
    if (st != SVDP_OK) return st;
    if (x == nullptr || y == nullptr || bad_batch(B) || !aligned16(x) || !aligned16(y)) return SVDP_ERR_INVALID_ARG;
    Workspace w;
    st = check_ws(layer, B, ws, ws_bytes, &w);
    if (st != SVDP_OK) return st;
    return dispatch(layer->wdtype, nb_of(B), [&](auto wt, auto nb) -> svdp_status {
        using W = typename decltype(wt)::type;
        constexpr int NB = decltype(nb)::value;
        if (!prepare_rows<W, NB, ROWS_DENSE>(layer)) return SVDP_ERR_UNSUPPORTED;
        return launch_rows<W, NB, ROWS_DENSE>(layer, x, B, nullptr, nullptr, nullptr, nullptr, nullptr, w, y,
                                              static_cast<hipStream_t>(stream));
    });
}

svdp_status svdp_ffn_step(const svdp_layer *layer, const void *x, int32_t B, float *y, uint64_t *mask_out,
                          int32_t *idx_out, int32_t *nnz_out, void *ws, size_t ws_bytes, void *stream)
{
    svdp_status st = check_layer(layer, true, true);
    if (st != SVDP_OK) return st;
    if (x == nullptr || y == nullptr || bad_batch(B) || !aligned16(x) || !aligned16(y)) return SVDP_ERR_INVALID_ARG;
    Workspace w;
    st = check_ws(layer, B, ws, ws_bytes, &w);
    if (st != SVDP_OK) return st;
    return step_impl(layer, x, B, y, mask_out, idx_out, nnz_out, w, static_cast<hipStream_t>(stream), nullptr);
}

svdp_status svdp_ffn_step_static(const svdp_layer *layer, const void *x, int32_t B, float *y, uint64_t *mask_out,
                                 int32_t *idx_out, int32_t *nnz_out, void *stream)
{
    svdp_status st = check_layer(layer, true, true);
    if (st != SVDP_OK) return st;
    if (x == nullptr || y == nullptr || bad_batch(B) || !aligned16(x) || !aligned16(y)) return SVDP_ERR_INVALID_ARG;
    if (!layer_fits(layer, nb_of(B))) return SVDP_ERR_UNSUPPORTED;
    // the size test comes first: a layer or batch beyond the array is refused whatever the device says
    if (carve(nullptr, layer->d, layer->D, layer->r, nb_of(B)).bytes > (size_t)SVDP_STATIC_SCRATCH_BYTES)
        return SVDP_ERR_WORKSPACE;
    void *scratch = static_scratch();
    if (scratch == nullptr) return SVDP_ERR_HIP;
    Workspace w;
    st = check_ws(layer, B, scratch, (size_t)SVDP_STATIC_SCRATCH_BYTES, &w);
    if (st != SVDP_OK) return st;
    return step_impl(layer, x, B, y, mask_out, idx_out, nnz_out, w, static_cast<hipStream_t>(stream), nullptr);
}

svdp_status svdp_ffn_step_glued(const svdp_layer *layer, const void *x_prev, const float *y_prev, const float *shift,
                                float eps, void *x_out, int32_t B, float *y, uint64_t *mask_out, int32_t *idx_out,
                                int32_t *nnz_out, void *ws, size_t ws_bytes, void *stream)
{
    svdp_status st = check_layer(layer, true, true);
    if (st != SVDP_OK) return st;
    if (x_prev == nullptr || y_prev == nullptr || shift == nullptr || x_out == nullptr || y == nullptr ||
        bad_batch(B) || !aligned16(x_prev) || !aligned16(x_out) || !aligned16(y) || !(eps >= 0.f))
        return SVDP_ERR_INVALID_ARG;
    Workspace w;
    st = check_ws(layer, B, ws, ws_bytes, &w);
    if (st != SVDP_OK) return st;
    const GlueArgs glue{y_prev, shift, eps, x_out};
    return step_impl(layer, x_prev, B, y, mask_out, idx_out, nnz_out, w, static_cast<hipStream_t>(stream), &glue);
}

svdp_status svdp_active_rows(const svdp_layer *layer, const void *x, int32_t B, const uint64_t *mask, float *y,
                             void *ws, size_t ws_bytes, void *stream)
{
    svdp_status st = check_layer(layer, false, true);
    if (st != SVDP_OK) return st;
    if (x == nullptr || mask == nullptr || bad_batch(B) || !aligned16(x) || (y != nullptr && !aligned16(y)))
        return SVDP_ERR_INVALID_ARG;
    Workspace w;
    st = check_ws(layer, B, ws, ws_bytes, &w);
    if (st != SVDP_OK) return st;
    return dispatch(layer->wdtype, nb_of(B), [&](auto wt, auto nb) -> svdp_status {
        using W = typename decltype(wt)::type;
        constexpr int NB = decltype(nb)::value;
        if (!prepare_rows<W, NB, ROWS_MASK>(layer)) return SVDP_ERR_UNSUPPORTED;
        hipStream_t hs = static_cast<hipStream_t>(stream);
        return launch_rows<W, NB, ROWS_MASK>(layer, x, B, mask, nullptr, nullptr, nullptr, nullptr, w, y, hs);
    });
}

svdp_status svdp_stack_glue(const void *x, const float *y, const float *shift, int32_t d, int32_t dtype, float eps,
                            void *x_next, void *stream)
{
    if (x == nullptr || y == nullptr || shift == nullptr || x_next == nullptr || d <= 0) return SVDP_ERR_INVALID_ARG;
    if (dtype != SVDP_F32 && dtype != SVDP_BF16) return SVDP_ERR_UNSUPPORTED;
    // whole 16-byte vectors of x, as for a layer's d
    if (d % (dtype == SVDP_BF16 ? 8 : 4) != 0) return SVDP_ERR_UNSUPPORTED;
    if (!aligned16(x) || !aligned16(y) || !aligned16(shift) || !aligned16(x_next)) return SVDP_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (dtype == SVDP_F32)
        launch(k_stack_glue<float>, dim3(1), dim3(256), 0, st, static_cast<const float *>(x), y, shift,
               d, eps, static_cast<float *>(x_next));
    else
        launch(k_stack_glue<bf16>, dim3(1), dim3(256), 0, st, static_cast<const bf16 *>(x), y, shift, d,
               eps, static_cast<bf16 *>(x_next));
    return hip_status(hipSuccess);
}

const char *svdp_status_string(svdp_status st)
{
    switch (st) {
    case SVDP_OK: return "ok";
    case SVDP_ERR_INVALID_ARG: return "invalid argument";
    case SVDP_ERR_UNSUPPORTED: return "unsupported shape or dtype";
    case SVDP_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case SVDP_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

size_t svdp_calib_workspace_bytes(int32_t D, int32_t T, int32_t eta)
{
    if (D < 1 || T < 1 || T > CAL_MAX_T || eta < 1) return 0;
    const size_t MS = ((size_t)T + eta - 1) / eta;
    return align_up((size_t)D * MS * 4) + 2 * align_up((size_t)D * (MS + 1) * 4) + align_up((size_t)D * 4) +
           align_up(sizeof(SelectState)) + align_up((size_t)SEL_BINS * 8) + 2 * align_up((size_t)D * 4);
}

int64_t svdp_calib_need(double sparsity, int32_t D, int32_t T)
{
    if (D < 1 || T < 1 || std::isnan(sparsity)) return -1;
    const int64_t all = (int64_t)D * (int64_t)T;
    const double target = sparsity * (double)D * (double)T;         // (sparsity * D) * T, in double
    if (!(target > 0.0)) return 0;
    if (target >= (double)all) return all;
    int64_t n = (int64_t)std::ceil(target);
    while (n > 0 && (double)(n - 1) >= target) --n;
    return n < 0 ? 0 : n > all ? all : n;
}

svdp_status svdp_calib_bias(const float *w, const float *s, int32_t D, int32_t T, int32_t eta, int64_t need,
                            float *b, int32_t *k, int32_t *steps, float *kendall, void *ws, size_t ws_bytes,
                            void *stream)
{
    if (w == nullptr || s == nullptr || b == nullptr || D < 1 || T < 1 || eta < 1 || need < 0)
        return SVDP_ERR_INVALID_ARG;
    if (T > CAL_MAX_T) return SVDP_ERR_UNSUPPORTED;
    const size_t bytes = svdp_calib_workspace_bytes(D, T, eta);
    if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & (ALIGN - 1)) || ws_bytes < bytes) return SVDP_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int MS = (T + eta - 1) / eta;
    char *p = static_cast<char *>(ws);
    float *key = reinterpret_cast<float *>(p);
    p += align_up((size_t)D * MS * 4);
    int32_t *drop = reinterpret_cast<int32_t *>(p);
    p += align_up((size_t)D * (MS + 1) * 4);
    float *tauc = reinterpret_cast<float *>(p);
    p += align_up((size_t)D * (MS + 1) * 4);
    int32_t *k0 = reinterpret_cast<int32_t *>(p);
    p += align_up((size_t)D * 4);
    SelectWork *work = reinterpret_cast<SelectWork *>(p);
    static_assert(sizeof(SelectWork) <= ALIGN, "the slot that the workspace keeps for the selection's state");
    p += align_up(sizeof(SelectState));
    long long *hist = reinterpret_cast<long long *>(p);
    p += align_up((size_t)SEL_BINS * 8);
    int32_t *lo = reinterpret_cast<int32_t *>(p);
    uint16_t *drop0 = reinterpret_cast<uint16_t *>(p);           // before the bounds: dropped pairs at the start
    static_assert(CAL_MAX_T < 1 << 16, "drop0");
    p += align_up((size_t)D * 4);
    int32_t *up = reinterpret_cast<int32_t *>(p);
    int n2 = 1;
    while (n2 < T) n2 <<= 1;
    auto sort = [&](auto per) {
        constexpr int PER = decltype(per)::value;
        const size_t lds = calib_sort_lds<PER>(n2, MS);
        if (!grant_lds<k_calib_sort<PER>>(lds)) return SVDP_ERR_UNSUPPORTED;
        launch(k_calib_sort<PER>, dim3(D), dim3(CAL_THREADS), lds, st, w, s, T, n2, eta, MS, key, drop, tauc, k0,
               drop0, kendall, reinterpret_cast<uint32_t *>(hist), SEL_BINS * 2, &work->readers, steps);
        return hip_status(hipSuccess);
    };
    svdp_status e = T <= 2 * CAL_THREADS ? sort(std::integral_constant<int, 2>{})
                    : T <= 4 * CAL_THREADS ? sort(std::integral_constant<int, 4>{})
                    : T <= 8 * CAL_THREADS ? sort(std::integral_constant<int, 8>{})
                                           : sort(std::integral_constant<int, 16>{});
    if (e != SVDP_OK) return e;
    const size_t items = (size_t)D * MS;
    const int hb = (int)std::min<size_t>((items + 256 * SEL_RUN - 1) / (256 * SEL_RUN), 256);       // more of them only meet at the counters
    // Two buffers of counts: `hist` and `up`, which is free until the bounds; where that is too small all pairs together
    // (D T < 512 * 4096) fit 32 bits, and both lie in `hist`.
    auto select = [&](auto *first, auto *second) {
        using Bin = std::remove_pointer_t<decltype(first)>;
        launch((k_select_hist<23, 8, -1, Bin>), dim3(hb), dim3(256), 0, st, key, drop, drop0, D, MS, (long long)need, 0,
               work, second, first);
        launch((k_select_hist<15, 8, 23, Bin>), dim3(hb), dim3(256), 0, st, key, drop, drop0, D, MS, (long long)need, 0, work,
               first, second);
        launch((k_select_hist<7, 8, 15, Bin>), dim3(hb), dim3(256), 0, st, key, drop, drop0, D, MS, (long long)need, 1, work,
               second, first);
        launch((k_select_hist<0, 7, 7, Bin>), dim3(hb), dim3(256), 0, st, key, drop, drop0, D, MS, (long long)need, 2, work,
               first, second);
        launch(k_select_last<Bin>, dim3(1), dim3(64), 0, st, work, second);
    };
    static_assert(CAL_MAX_T <= 4096 && SEL_BINS * 8 <= 512 * 4, "see above");
    if (D >= 512) {
        select(hist, reinterpret_cast<long long *>(up));
    } else {
        uint32_t *h32 = reinterpret_cast<uint32_t *>(hist);
        select(h32, h32 + SEL_BINS);
    }
    const SelectState *state = &work->state[SEL_STATES - 1];
    // the digit counts are done with: their place holds the blocks' gains, so there are at most SEL_BINS blocks
    const int chunk = (int)(((long long)D + 256 * SEL_BINS - 1) / (256 * SEL_BINS)) * 256, blocks = (D + chunk - 1) / chunk;
    launch(k_select_bounds, dim3(blocks), dim3(256), 0, st, key, drop, D, MS, chunk, state, lo, up, hist);
    launch(k_select_finish, dim3(blocks), dim3(256), 0, st, lo, up, drop, tauc, k0, D, T, eta, MS, chunk, state, hist,
           b, k, steps);
    return hip_status(hipSuccess);
}

size_t svdp_calib_stats_workspace_bytes(const svdp_layer *layer, int32_t T)
{
    if (check_layer(layer, true, true) != SVDP_OK || layer->wdtype != SVDP_BF16 || T < 1) return 0;
    return align_up((size_t)layer->r * layer->d * 2) + align_up((size_t)layer->D * 4) +
           align_up((size_t)T * 3 * layer->r * 2);
}

svdp_status svdp_calib_stats(const svdp_layer *layer, const void *X, int32_t T, float *w, float *s, void *ws,
                             size_t ws_bytes, void *stream)
{
    svdp_status e = check_layer(layer, true, true);
    if (e != SVDP_OK) return e;
    if (X == nullptr || w == nullptr || s == nullptr || T < 1) return SVDP_ERR_INVALID_ARG;
    if (layer->wdtype != SVDP_BF16) return SVDP_ERR_UNSUPPORTED;
    const size_t bytes = svdp_calib_stats_workspace_bytes(layer, T);
    if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & (ALIGN - 1)) || ws_bytes < bytes) return SVDP_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int d = layer->d, D = layer->D, r = layer->r;
    char *p = static_cast<char *>(ws);
    bf16 *Pt = reinterpret_cast<bf16 *>(p);                      // [r][d]
    p += align_up((size_t)r * d * 2);
    float *cn = reinterpret_cast<float *>(p);                    // [D] squared column norms of W_down
    p += align_up((size_t)D * 4);
    uint16_t *tp = reinterpret_cast<uint16_t *>(p);              // [T][3r]: t = x P as three bf16 terms
    const bf16 *Wg = static_cast<const bf16 *>(layer->W_gate), *Wu = static_cast<const bf16 *>(layer->W_up);
    const bf16 *Xb = static_cast<const bf16 *>(X);
    auto tiles = [](int n, int b) { return (n + b - 1) / b; };

    if (!grant_lds<k_gemm_wide>(GW_LDS)) return SVDP_ERR_UNSUPPORTED;
    launch(k_transpose16, dim3(tiles(r, 32), tiles(d, 32)), dim3(256), 0, st,
           static_cast<const uint16_t *>(layer->P), d, r, reinterpret_cast<uint16_t *>(Pt));
    // t = X P, split into three terms.  Its tiles alone are few (32 at r = 256, T = 2048: 90 us on an eighth of the chip,
    // 16 + 5 us in eight parts), so they are cut along K into as many parts as fill it; the parts meet in s, which the
    // last launch overwrites.
    const int t_tiles = tiles(r, GM_BN) * tiles(T, GM_BM);
    const int parts = std::max(1, std::min({256 / t_tiles, d / 256, D / r, 16}));
    const int kpart = round_up(tiles(d, parts), GM_BK), nz = tiles(d, kpart);
    const NormJob norm{static_cast<const bf16 *>(layer->W_downT), D, d, cn};
    const int nx = tiles(r, GM_BN), ny = tiles(T, GM_BM), norm_blocks = tiles(D, NORM_ROWS);
    if (nz > 1) {
        launch((k_gemm_nt<EPI_PLAIN>), dim3(nx * ny * nz + norm_blocks), dim3(GM_THREADS), 0, st, Xb, d, Pt, d, T, r, d,
               s, nullptr, r, kpart, nx, ny, nz, norm);
        launch(k_sum_split3, dim3(tiles(T * r, 256)), dim3(256), 0, st, s, nz, T, r, tp);
    } else {
        launch((k_gemm_nt<EPI_SPLIT3>), dim3(nx * ny + norm_blocks), dim3(GM_THREADS), 0, st, Xb, d, Pt, d, T, r, d,
               nullptr, tp, 3 * r, d, nx, ny, 1, norm);
    }
    // w = (ReLU(W_gate X^T) * (W_up X^T))^2 * cn and s = Q t^T over the three terms
    const bf16 *Qb = static_cast<const bf16 *>(layer->Q), *tb = reinterpret_cast<const bf16 *>(tp);
    const WideJob jw = wide_job(Wg, Wu, d, d, Xb, d, D, T, d, cn, w, T), js = wide_job(Qb, nullptr, r, r, tb, 3 * r, D, T, 3 * r,
                                                                                      nullptr, s, T);
    launch(k_gemm_wide, dim3(jw.tiles + js.tiles), dim3(GW_THREADS), GW_LDS, st, jw, js);
    return hip_status(hipSuccess);
}

size_t svdp_whiten_workspace_bytes(int32_t d, int32_t D, int32_t T, int32_t r)
{
    if (d < 64 || d % 64 != 0 || D < 1 || T < d || r < 1 || r > d) return 0;
    return whiten_ws_bytes(d, D, T, r);
}

svdp_status svdp_whiten_factors(const void *W_gate, const void *X, int32_t d, int32_t D, int32_t T, int32_t r,
                                int32_t wdtype, float *P, float *Q, float *sigma, int32_t *sweeps, void *ws,
                                size_t ws_bytes, void *stream)
{
    if (W_gate == nullptr || X == nullptr || P == nullptr || Q == nullptr || d < 1 || D < 1 || T < 1 || r < 1)
        return SVDP_ERR_INVALID_ARG;
    if (wdtype != SVDP_F32 && wdtype != SVDP_BF16) return SVDP_ERR_UNSUPPORTED;
    if (d < 64 || d % 64 != 0 || T < d || r > d) return SVDP_ERR_UNSUPPORTED;
    if (ws == nullptr || (reinterpret_cast<uintptr_t>(ws) & (ALIGN - 1))) return SVDP_ERR_WORKSPACE;
    const WhitenWs w = carve_whiten(ws, d, D, T, r);
    if (ws_bytes < w.bytes || !w.fits) return SVDP_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (wdtype == SVDP_F32) return whiten_impl<float>(W_gate, X, d, D, T, r, P, Q, sigma, sweeps, w, st);
    return whiten_impl<bf16>(W_gate, X, d, D, T, r, P, Q, sigma, sweeps, w, st);
}

const char *svdp_version(void) { return "0.5"; }

}  // extern "C"
