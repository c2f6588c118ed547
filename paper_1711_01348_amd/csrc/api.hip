// Device entry points of the C ABI: dispatch on the kernel family chosen at plan time.
#include <hip/hip_runtime.h>

#include <mutex>

#include "launch.h"

using namespace tad;

// Scratch memory of tad_eval_backward_static: one array per GPU, part of the loaded code object, held until the
// process ends.  In host code the array's name only stands for the symbol; its device address is looked up once per
// device with hipGetSymbolAddress and that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[TAD_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];

int static_scratch(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TAD_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TAD_EDEVICE;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return TAD_OK;
}
// Paths that keep 64-bit values or whole vectors in the workspace; with a smaller or oddly aligned one, or none, the family's
// kernels run.
bool room(const tad_plan &pl, const void *ws, size_t ws_bytes) {
    return pl.ws_full == 0 || (ws && ws_bytes >= pl.ws_full && (reinterpret_cast<uintptr_t>(ws) & 15) == 0);
}
// The products to run in this workspace, or null.
const ProductSet *products_in(const tad_plan &pl, const ProductSet &set, const ProductSet *lean, const void *ws, size_t ws_bytes) {
    if (room(pl, ws, ws_bytes)) return &set;
    return lean && ws && ws_bytes >= pl.ws_lean && (reinterpret_cast<uintptr_t>(ws) & 15) == 0 ? lean : nullptr;
}
const ProductSet *use_product(const tad_plan &pl, const void *ws, size_t ws_bytes) {
    if (!pl.prod.on) return nullptr;
    if (pl.prod.set.ws_bytes == 0) return &pl.prod.set;
    return products_in(pl, pl.prod.set, pl.prod.lean_on ? &pl.prod.lean : nullptr, ws, ws_bytes);
}
const ProductSet *use_separable(const tad_plan &pl, const void *ws, size_t ws_bytes) {
    return pl.sep.on ? products_in(pl, pl.sep.set, pl.sep.lean_on ? &pl.sep.lean : nullptr, ws, ws_bytes) : nullptr;
}
bool use_worked_wide(const tad_plan &pl, const void *ws, size_t ws_bytes) { return pl.worked_wide && room(pl, ws, ws_bytes); }
bool use_pattern_wide(const tad_plan &pl, const void *ws, size_t ws_bytes) {
    return pl.pattern_wide != TAD_FAMILY_GENERIC && room(pl, ws, ws_bytes);
}
}  // namespace

extern "C" {

int tad_eval_forward(const tad_plan *plan, const void *const *args_dev, void *f_dev, void *ws_dev,
                     size_t ws_bytes, void *stream) {
    if (!plan || !args_dev || !f_dev) return TAD_EINVAL;
    for (size_t p = 0; p < plan->args.size(); ++p)
        if (!args_dev[plan->root[p]]) return TAD_EINVAL;
    if (plan->ws_bytes && (!ws_dev || ws_bytes < plan->ws_bytes)) return TAD_ENOMEM;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (plan->sep.forward_on)
        if (const ProductSet *set = use_separable(*plan, ws_dev, ws_bytes)) return separable_forward(*plan, *set, args_dev, f_dev, ws_dev, s);
    if (use_worked_wide(*plan, ws_dev, ws_bytes)) return worked_wide_forward(*plan, args_dev, f_dev, s);
    if (use_pattern_wide(*plan, ws_dev, ws_bytes)) return pattern_wide_forward(*plan, args_dev, f_dev, s);
    if (plan->window.on) return window_forward(*plan, args_dev, f_dev, s);
    if (plan->prod.forward_on)
        if (const ProductSet *set = use_product(*plan, ws_dev, ws_bytes)) return product_forward(*plan, *set, args_dev, f_dev, ws_dev, s);
    switch (plan->fwd_family) {
    case TAD_FAMILY_GENERIC: return generic_forward(*plan, args_dev, f_dev, ws_dev, s);
    case TAD_FAMILY_WORKED: return worked_forward(*plan, args_dev, f_dev, s);
    case TAD_FAMILY_WORKED_MFMA: return mfma_forward(*plan, args_dev, f_dev, ws_dev, plan->mfma_split && room(*plan, ws_dev, ws_bytes), s);
    case TAD_FAMILY_ROW_REDUCE:
    case TAD_FAMILY_DIAGONAL:
    case TAD_FAMILY_ANTIDIAGONAL: return pattern_forward(*plan, args_dev, f_dev, s);
    case TAD_FAMILY_STRIDED: return strided_forward(*plan, args_dev, f_dev, s);
    case TAD_FAMILY_CONTRACTION: return contract_forward(*plan, args_dev, f_dev, ws_dev, plan->split && room(*plan, ws_dev, ws_bytes), s);
    case TAD_FAMILY_PROGRAM: return program_forward(*plan, args_dev, f_dev, ws_dev, s);
    default: return TAD_EUNSUPPORTED;
    }
}

int tad_eval_backward(const tad_plan *plan, const void *const *args_dev, const void *f_dev,
                      const void *df_dev, void *const *dx_dev, void *ws_dev, size_t ws_bytes, void *stream) {
    if (!plan || !args_dev || !f_dev || !df_dev || !dx_dev) return TAD_EINVAL;
    for (size_t p = 0; p < plan->args.size(); ++p) {
        if (!args_dev[plan->root[p]]) return TAD_EINVAL;
        if (dx_dev[p] && (!plan->ap[p].derived || plan->root[p] != (int)p)) return TAD_EINVAL;  // not planned / alias
    }
    if (plan->ws_bytes && (!ws_dev || ws_bytes < plan->ws_bytes)) return TAD_ENOMEM;
    hipStream_t s = static_cast<hipStream_t>(stream);
    bool any_wanted = false;
    for (size_t p = 0; p < plan->args.size(); ++p) any_wanted |= dx_dev[p] != nullptr;
    if (!any_wanted) return TAD_OK;
    if (const ProductSet *set = use_separable(*plan, ws_dev, ws_bytes)) return separable_backward(*plan, *set, args_dev, f_dev, df_dev, dx_dev, ws_dev, s);
    if (use_worked_wide(*plan, ws_dev, ws_bytes)) return worked_wide_backward(*plan, args_dev, f_dev, df_dev, dx_dev, ws_dev, s);
    if (plan->pattern_wide_sums && use_pattern_wide(*plan, ws_dev, ws_bytes)) return pattern_wide_backward(*plan, args_dev, df_dev, dx_dev, ws_dev, s);
    if (plan->window.on && room(*plan, ws_dev, ws_bytes)) return window_backward(*plan, args_dev, df_dev, dx_dev, ws_dev, s);
    void *rest[kMaxArgs];   // the gradients the dense products leave to the family
    if (const ProductSet *set = use_product(*plan, ws_dev, ws_bytes)) {
        for (size_t p = 0; p < plan->args.size(); ++p) rest[p] = dx_dev[p];
        const int rc = product_backward(*plan, *set, args_dev, df_dev, rest, ws_dev, s);
        if (rc) return rc;
        dx_dev = rest;
        any_wanted = false;
        for (size_t p = 0; p < plan->args.size(); ++p) any_wanted |= rest[p] != nullptr;
        if (!any_wanted) return TAD_OK;
    }
    // a specialised family owns all gradients of its expression; anything left is generic
    int fam = TAD_FAMILY_GENERIC;
    for (size_t p = 0; p < plan->args.size(); ++p)
        if (plan->ap[p].derived && plan->ap[p].family != TAD_FAMILY_GENERIC) fam = plan->ap[p].family;
    switch (fam) {
    case TAD_FAMILY_GENERIC: return generic_backward(*plan, args_dev, f_dev, df_dev, dx_dev, ws_dev, s);
    case TAD_FAMILY_WORKED: return worked_backward(*plan, args_dev, f_dev, df_dev, dx_dev, ws_dev, s);
    case TAD_FAMILY_WORKED_MFMA: return mfma_backward(*plan, args_dev, f_dev, df_dev, dx_dev, ws_dev, plan->mfma_split && room(*plan, ws_dev, ws_bytes), s);
    case TAD_FAMILY_ROW_REDUCE:
    case TAD_FAMILY_DIAGONAL:
    case TAD_FAMILY_ANTIDIAGONAL: return pattern_backward(*plan, args_dev, df_dev, dx_dev, ws_dev, s);
    case TAD_FAMILY_STRIDED: return strided_backward(*plan, args_dev, f_dev, df_dev, dx_dev, ws_dev, s);
    case TAD_FAMILY_CONTRACTION: return contract_backward(*plan, args_dev, df_dev, dx_dev, ws_dev, plan->split && room(*plan, ws_dev, ws_bytes), s);
    case TAD_FAMILY_PROGRAM: return program_backward(*plan, args_dev, f_dev, df_dev, dx_dev, ws_dev, s);
    default: return TAD_EUNSUPPORTED;
    }
}

int tad_eval_backward_static(const tad_plan *plan, const void *const *args_dev, const void *f_dev,
                             const void *df_dev, void *const *dx_dev, void *stream) {
    if (!plan) return TAD_EINVAL;
    if (plan->ws_bytes > (size_t)TAD_STATIC_SCRATCH_BYTES) return TAD_ENOMEM;
    void *ws = nullptr;
    int rc = static_scratch(&ws);
    if (rc != TAD_OK) return rc;
    // the kernels write every workspace entry before they read it, so the contents the previous call left behind
    // need no clearing
    return tad_eval_backward(plan, args_dev, f_dev, df_dev, dx_dev, ws, TAD_STATIC_SCRATCH_BYTES, stream);
}

}  // extern "C"
