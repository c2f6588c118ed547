// The element-wise function a product applies to its results.
#pragma once
#include "launch.h"
#include "prog_eval.h"

namespace tad {

// What becomes of a sum s before it is stored (the outer function of an expression, or g = df * its derivative).
struct ProductOuter {
    DevProg prog;          // has a register form
    ArgPtrs args;          // operands the program reads, null for the others
    int64_t off_r[kMaxArgs], off_c[kMaxArgs];   // their element offsets along the rows and columns of the result
    const void *df;        // null: c = prog(s), else c = df * prog(s)
    void *s_out;           // null, or where s goes as well
};

}  // namespace tad
