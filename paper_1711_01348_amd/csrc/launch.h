// Declarations shared by the kernel translation units and the C ABI front end.
#pragma once
#include <hip/hip_runtime.h>

#include "plan.hpp"

namespace tad {

struct ArgPtrs {
    const void *p[kMaxArgs];
};

int generic_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
int generic_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                     void *const *dx, void *ws, hipStream_t s);

int worked_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int worked_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                    void *const *dx, void *ws, hipStream_t s);

// worked expression in either precision, rows of any length, K <= 16: sums in 64 bits
int worked_wide_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int worked_wide_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df, void *const *dx, void *ws, hipStream_t s);

int mfma_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
int mfma_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df, void *const *dx,
                  void *ws, hipStream_t s);
int pattern_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int pattern_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws,
                     hipStream_t s);

int strided_forward(const tad_plan &pl, const void *const *args, void *f, hipStream_t s);
int strided_backward(const tad_plan &pl, const void *const *args, const void *f, const void *df,
                     void *const *dx, void *ws, hipStream_t s);

int contract_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
int contract_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws,
                      hipStream_t s);

// Sums of products as dense products.  product_backward writes the gradients it is responsible for and clears their
// entries of dx; the rest is left to the family's kernels.
int product_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
int product_backward(const tad_plan &pl, const void *const *args, const void *df, void **dx, void *ws, hipStream_t s);

// one product; a64, b64, c64: 64-bit elements; ws: partial sums of shared tiles
int product_run(const ProductDesc &d, const void *a, bool a64, const void *b, bool b64, void *c, bool c64, void *ws, hipStream_t s);

// sums of products of two functions (separable.hpp)
int separable_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
int separable_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws, hipStream_t s);

int program_forward(const tad_plan &pl, const void *const *args, void *f, void *ws, hipStream_t s);
int program_backward(const tad_plan &pl, const void *const *args, const void *df, void *const *dx, void *ws,
                     hipStream_t s);

}  // namespace tad
