// Index-notation front-end and leaf generator (host side).
//
// A statement of tensor index notation (Sec. II-A) over Dense/Compressed
// operands is parsed, given a concordant loop order (each sparse operand's
// levels iterated outer to inner, Sec. IV-C), and lowered to a loop nest in
// which every index variable is either a coordinate-value loop (a dense
// range) or a merge over the positions of the Compressed levels that index
// it (coordinate-position loops, co-iterated: intersection for products,
// union for sums; Sec. IV-C).  The nest is emitted as HIP source, compiled
// at run time for gfx950 and launched one thread per coordinate of the
// outermost index; CSR outputs of CSR operands are counted and filled with
// the rows of a workgroup staged in LDS.  Outputs: a dense tensor (every entry written), a scalar,
// or a CSR matrix assembled in two phases (count, scan, fill; Sec. V-B).
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <memory>
#include <string>
#include <vector>

#include "spleaf.h"

namespace spl {
namespace tin {

enum OutKind { kOutDense = 0, kOutScalar = 1, kOutCsr = 2 };

// One operand of a statement as the caller binds it: exactly one of
// sparse / dense is set.
struct Binding {
    std::string name;
    const spl_sparse *sparse = nullptr;
    const spl_dense *dense = nullptr;
};

// One kernel-argument slot: what the host writes into it.
struct Slot {
    enum Kind { kRows, kExtent, kPos, kCrd, kVals, kDenseData, kDenseLd, kLevelDim,
                kOutData, kOutLd, kOutPos, kOutCrd, kOutVals, kPartials, kScratch, kPool } kind;
    int operand = -1;  // index into the bindings (right side), -1 for the output
    int level = 0;     // sparse level, or the variable for kExtent
};

// A planned and generated statement for one set of operand formats.
struct Program {
    std::string key;
    std::string source;
    int out_kind = kOutDense;
    int vtype = SPL_F64;          // value type of every operand and the output
    int64_t rows = 0;             // extent of the outermost index (threads)
    int64_t out_cols = 1;         // dense output: entries per outermost coordinate
    std::vector<int64_t> extents; // per index variable, from this call's operands
    bool scratch_rows = false;    // dense F32 output accumulated in an F64 scratch
    bool stages = false;          // the count and fill kernels can stage rows in LDS
    std::vector<int> staged_ops;  // the operand of every access staged then
    int entry_bytes = 0;          // LDS bytes of a staged output entry
    std::vector<Slot> slots;
    hipModule_t module = nullptr;
    hipFunction_t f_eval = nullptr, f_count = nullptr, f_fill = nullptr;
    ~Program();
};

// Parse `stmt`, check it against the bindings and plan the loop nest.
// `out` is the left side's binding (its sparse/dense pointers may hold
// placeholders: only formats, dtypes and dimensions are read here).
// source: generate prog.source too (a call whose leaves are compiled already
// needs the plan alone).  Returns SPL_OK or a status with the reason in `err`.
spl_status plan(const char *stmt, const std::vector<Binding> &ops, const Binding &out,
                bool source, Program &prog, std::string &err);

// Compile prog.source with hiprtc for gfx950 and load it on the current
// device.
spl_status compile(Program &prog, std::string &err);

// Kernel-argument slots for one call (64-bit each, in the order of
// prog.slots).  `out` as bound for this call; `partials` and `scratch` are
// device workspace pointers (may be null when unused); `pool` is the launch's
// dynamic LDS (stage_shape).
void fill_slots(const Program &prog, const std::vector<Binding> &ops, const Binding &out,
                const int32_t *out_pos, void *partials, void *scratch, unsigned pool,
                std::vector<unsigned long long> &slots);

// Rows (threads) per workgroup and dynamic LDS bytes of a launch of the count
// (out_nnz < 0) or fill kernel: room for the runs of its rows at the
// operands' mean row lengths and a quarter as much again.  A workgroup whose runs
// do not fit walks them in HBM; when not even 64 mean rows fit, all do
// (256 threads, no LDS).
// 128 rows: the sum of two matrices of 1e6 rows and 8 entries a row takes
// 228 us a call, 239 with 256 rows and 228 with 64.
constexpr unsigned kStageRows = 128;
constexpr unsigned kStageBytes = 65536;  // dynamic LDS every launch may ask for
constexpr unsigned kStageSlack = 1024;   // short runs vary more than their mean
constexpr double kStageSpread = 1.25;
void stage_shape(const Program &prog, const std::vector<Binding> &ops, int64_t out_nnz,
                 unsigned &block, unsigned &pool);

// Workspace bytes a call of `prog` needs (partials, F64 row scratch, scan
// space for the symbolic phase), at 256-byte granularity.
size_t workspace_bytes(const Program &prog, bool symbolic);

}  // namespace tin
}  // namespace spl
