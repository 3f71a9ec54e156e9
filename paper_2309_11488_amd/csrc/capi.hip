// C ABI of the BCSR BiCGStab-ILU0 library: handles, validation, device
// buffers and the host side of the solve (kernel sequencing and the
// convergence poll).  All arithmetic of the path runs in kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <fstream>
#include <map>
#include <memory>
#include <mutex>
#include <sstream>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/rsolve.h"
#include "analysis.h"
#include "kernels.h"

using rs::DevSchedule;
using rs::Krylov;
using rs::SysState;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string &msg) {
    g_err = msg;
    return code;
}

#define HIP_TRY(expr)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return fail(e_ == hipErrorOutOfMemory ? RS_OUT_OF_MEMORY : RS_HIP_ERROR,               \
                        std::string(#expr) + ": " + hipGetErrorString(e_));                        \
    } while (0)

// Pattern fingerprint: FNV-1a style over 32-bit words in four independent
// lanes (a pattern of a million rows hashes in a few milliseconds).
uint64_t pattern_fingerprint(const std::vector<int32_t> &rp, const std::vector<int32_t> &ci) {
    const uint64_t prime = 1099511628211ull;
    uint64_t h[4] = {1469598103934665603ull, 0x9e3779b97f4a7c15ull, 0xc2b2ae3d27d4eb4full, 0x165667b19e3779f9ull};
    auto mix = [&](const std::vector<int32_t> &v) {
        const size_t n = v.size(), n4 = n & ~(size_t)3;
        for (size_t i = 0; i < n4; i += 4)
            for (int l = 0; l < 4; ++l) h[l] = (h[l] ^ (uint32_t)v[i + l]) * prime;
        for (size_t i = n4; i < n; ++i) h[0] = (h[0] ^ (uint32_t)v[i]) * prime;
        h[1] = (h[1] ^ n) * prime;
    };
    mix(rp);
    mix(ci);
    uint64_t r = h[0];
    for (int l = 1; l < 4; ++l) r = (r ^ h[l]) * prime;
    return r;
}

// Device allocation owned by a handle.
struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
    ~DevBuf() { if (p) (void)hipFree(p); }
    hipError_t alloc(size_t b) {
        if (p && bytes >= b) return hipSuccess;
        if (p) (void)hipFree(p);
        p = nullptr;
        bytes = 0;
        // 64 spare bytes: row kernels copy whole 16-byte units into LDS and
        // may read up to 15 bytes past the last block of an array
        b += 64;
        hipError_t e = hipMalloc(&p, b);
        if (e == hipSuccess) bytes = b;
        return e;
    }
    template <typename T> T *as() const { return (T *)p; }
};

// Stream-ordered upload of a host array the handle owns (the caller
// synchronises `s` before the data is used on another stream).
hipError_t upload(DevBuf &buf, const std::vector<int32_t> &v, hipStream_t s) {
    hipError_t e = buf.alloc(v.size() * sizeof(int32_t));
    if (e != hipSuccess || v.empty()) return e;
    return hipMemcpyAsync(buf.p, v.data(), v.size() * sizeof(int32_t), hipMemcpyHostToDevice, s);
}

// Process-wide and not thread-safe; off unless enabled.
// Optional per-class kernel timing with HIP events recorded on the launch
// stream around each unit of work (a kernel launch, or a whole sweep).  The
// SpMV classes are split so that v = A phat, which runs in every launched
// iteration, can be timed apart from t = A shat, which exits early in an
// iteration that stopped at its half step.
enum ProfClass {
    PC_FACTOR = 0, PC_LSWEEP = 1, PC_USWEEP = 2, PC_SPMV_V = 3, PC_VEC = 4, PC_SPMV_T = 5, PC_GM = 6,
    PC_APPLY = 7, PC_COUNT = 8
};

struct Prof {
    int mask = 0;
    double ms[PC_COUNT] = {}, bytes[PC_COUNT] = {};
    long long units[PC_COUNT] = {};
    struct Pending {
        int cls;
        hipEvent_t a, b;
        double bytes;
    };
    std::vector<Pending> pending;
    std::vector<hipEvent_t> pool;
};
Prof g_prof;

hipEvent_t prof_event() {
    hipEvent_t e = nullptr;
    if (!g_prof.pool.empty()) {
        e = g_prof.pool.back();
        g_prof.pool.pop_back();
    } else if (hipEventCreate(&e) != hipSuccess) {
        e = nullptr;
    }
    return e;
}

// Records an event pair on the stream around the scope.  With `dispatch`,
// the events are instead handed to the single kernel launch inside the scope
// (start(), stop()), which records them itself at the kernel's start and
// end, so the time excludes the launch.
struct ProfScope {
    int cls;
    hipStream_t s;
    double bytes;
    bool dispatch;
    hipEvent_t a = nullptr, b = nullptr;
    ProfScope(int c, hipStream_t st, double by, bool disp = false, bool on = true)
        : cls(c), s(st), bytes(by), dispatch(disp) {
        if (on && ((g_prof.mask >> cls) & 1)) {
            a = prof_event();
            if (a && dispatch) {
                b = prof_event();
                if (!b) a = nullptr;
            } else if (a) {
                (void)hipEventRecord(a, s);
            }
        }
    }
    hipEvent_t start() const { return a; }
    hipEvent_t stop() const { return b; }
    ~ProfScope() {
        if (!a) return;
        if (!dispatch) {
            b = prof_event();
            if (!b) return;
            (void)hipEventRecord(b, s);
        }
        g_prof.pending.push_back({cls, a, b, bytes});
    }
};

void prof_flush() {
    for (auto &p : g_prof.pending) {
        float ms = 0.f;
        if (hipEventSynchronize(p.b) == hipSuccess && hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
            g_prof.ms[p.cls] += ms;
            g_prof.units[p.cls] += 1;
            g_prof.bytes[p.cls] += p.bytes;
        }
        g_prof.pool.push_back(p.a);
        g_prof.pool.push_back(p.b);
    }
    g_prof.pending.clear();
}

}  // namespace

struct rs_bcsr {
    int n = 0, nnzb = 0, batch = 1;
    int spmv_variant = rs::RV_W4_LDS;
    uint64_t hash = 0;
    std::vector<int32_t> h_rowptr, h_colidx;
    DevBuf rowptr, colidx, vals;
    // standard wells kept separate (bcsr_set_wells), caller numbering
    int nw = 0, np = 0;
    long long wells_version = 0;
    std::vector<int32_t> h_well_ptr, h_perf_row, h_row_ptr, h_row_perf, h_perf_well;
    DevBuf w_well_ptr, w_perf_row, w_row_ptr, w_row_perf, w_perf_well, w_B, w_C, w_Dinv, w_t2;
    // the wells as the caller-order SpMVs see them, systems from `first`
    rs::WellsDev wells(int first = 0) const {
        rs::WellsDev w;
        if (nw == 0) return w;
        w.nw = nw; w.np = np;
        w.well_ptr = w_well_ptr.as<int32_t>(); w.perf_x = w_perf_row.as<int32_t>();
        w.row_ptr = w_row_ptr.as<int32_t>(); w.row_perf = w_row_perf.as<int32_t>();
        w.perf_well = w_perf_well.as<int32_t>();
        w.B = w_B.as<double>() + (size_t)first * np * 12; w.C = w_C.as<double>() + (size_t)first * np * 12;
        w.Dinv = w_Dinv.as<double>() + (size_t)first * nw * 16; w.t2 = w_t2.as<double>() + (size_t)first * nw * 4;
        return w;
    }
};

// Rows' perforation lists: row_ptr (n + 1) and row_perf, perforations of a
// row ascending; rows given by row_of[p].
static void perforation_index(int n, const std::vector<int32_t> &row_of, std::vector<int32_t> &row_ptr,
                              std::vector<int32_t> &row_perf) {
    row_ptr.assign((size_t)n + 1, 0);
    for (int32_t r : row_of) row_ptr[r + 1]++;
    for (int i = 0; i < n; ++i) row_ptr[i + 1] += row_ptr[i];
    row_perf.assign(row_of.size(), 0);
    std::vector<int32_t> next(row_ptr.begin(), row_ptr.end() - 1);
    for (size_t p = 0; p < row_of.size(); ++p) row_perf[next[row_of[p]]++] = (int32_t)p;
}

// The analysis of one pattern: the host schedule and its device copy.
// Immutable once built; every preconditioner handle of the pattern holds a
// reference, and the last one to go frees it.
struct Analysis {
    uint64_t hash = 0;
    rs::Schedule sch;
    DevSchedule dev{};
    DevBuf perm, prow, pcol, psrc, lrows, lptr, lcol, lsrc, ldq, l2u, upd_ptr, upd, urows, uptr, ucol, usrc, dsrc;
    DevBuf lsrc_a, usrc_a, dsrc_a, rest_dst, rest_src;
    DevBuf lt_start, ut_start, la_start, ua_start, ls_start, us_start;
    // U blocks of rows with lower blocks: with FP32 factors the only U the
    // factorisation keeps in FP64 (later levels' updates read it)
    double u_kept = 0;
};

struct rs_ilu0 {
    int n = 0, nnzb = 0, batch = 1;
    uint64_t hash = 0;
    std::shared_ptr<const Analysis> an;
    // factors
    int precision = -1;
    bool factored = false;
    DevBuf pvals, L, U, Dinv, Lf, Uf, Dinvf, bad;
    // what a call reads from the device, in one pinned block (a pageable copy
    // costs a step of 4 000 cells 8 us more): the states, the sweep counters
    // and the pivot record
    void *pinned = nullptr;
    SysState *h_state = nullptr;
    rs::SweepCtr *h_ctr = nullptr;
    int32_t *bad_host = nullptr;
    // the last application queued without a host wait: the next call may use
    // another stream, and works in the same buffers
    hipEvent_t ev_apply = nullptr;
    hipStream_t apply_stream = nullptr;   // its stream, only asked whether it is being captured
    bool apply_queued = false;
    // solve workspace
    DevBuf work, ywork, ywork2, ftickets, vpart, part, spart, fpart, tickets, state, bstage, xstage, ctrs, fctr;
    bool no_flow = false;      // no room for what one-launch applications need besides
    bool y_marked = false;     // ywork holds the mark everywhere (single-launch sweeps)
    Krylov k{};
    // GMRES workspace: Krylov basis, per-system cycle state, reduction partials
    DevBuf gm_basis, gm_state, gm_part, gm_vpart;
    int last_gm_steps = 1;
    int chunk = 1;
    bool predict = true;       // first poll after as many iterations as the last converged solve needed
    int last_iters = 1;
    int spin_limit = rs::kSpinLimitDefault;   // polls before a tile dependency wait gives up
    // device time of the last factorisation and of the current solve call
    hipEvent_t ev_f0 = nullptr, ev_f1 = nullptr, ev_s0 = nullptr, ev_s1 = nullptr;
    double factor_ms = 0.0;
    // RS_OPT_FACTOR_ASYNC: the last factorisation was queued and its result
    // not read yet (factor_status and bad_orig hold it once it is)
    bool factor_async = false, factor_pending = false;
    int factor_status = RS_OK;
    std::vector<int32_t> bad_orig;
    bool tile_sweeps = true;   // single-launch sweeps (else one launch per level)
    int sweep_grid = 1024;     // workgroups of a single-launch sweep
    int spmv_variant = rs::RV_W4_LDS;   // launch shape of the SpMVs
    int sweep_variant = rs::RV_W4_LDS;  // launch shape of the per-level sweeps
    int reduce_split = 0;               // RS_OPT_REDUCE_SPLIT
    bool fuse_spmv = true;              // RS_OPT_FUSE_SPMV
    bool y_input = true;                // RS_OPT_Y_INPUT
    bool lower_parts = true;            // RS_OPT_LOWER_PARTS
    DevBuf lpwork;                      // its two vectors (allocated on first use)
    // a pattern with fused rows: the factorisation stored no U of the
    // factor type for those rows (their fused upper launches read A'); it is
    // filled from A' when a consumer of U needs it (single-launch sweeps,
    // per-level sweeps of FP32 factors outside the fused iteration,
    // ilu0_get_factors)
    bool u_missing = false;
    // the wells of the matrix last solved with, in the new numbering
    const rs_bcsr *wells_of = nullptr;
    long long wells_version = -1;
    std::vector<int32_t> h_wperf_x, h_wrow_ptr, h_wrow_perf;
    DevBuf wperf_x, wrow_ptr, wrow_perf, wt2, wfix;
    std::vector<int32_t> h_wfix;   // rows below fuse_n0 that a perforation couples
    rs::WellsDev wdev{};
    int split() const { return reduce_split; }
    // polled partials of the vector and of the GMRES kernels
    size_t vpart_stride() const { return 2 * (size_t)rs::vec_blocks(n); }
    size_t vpart_bytes() const { return (size_t)batch * vpart_stride() * sizeof(double); }
    size_t gm_vpart_bytes() const { return (size_t)batch * rs::gm_poll_stride() * sizeof(double); }
    // a BiCGStab iteration captured as HIP graphs, replayed on the caller's
    // stream: one segment per set of consecutive parts of the iteration (the
    // whole iteration, or the runs between the parts of a kernel class that
    // is being timed with events and so launched directly)
    bool use_graph = true;
    hipStream_t cap_stream = nullptr;
    // every setting a captured iteration depends on
    struct GraphKey {
        int precision = -1, tile_sweeps = 0, spmv_variant = 0, sweep_variant = 0, split = 0, sweep_grid = 0;
        int spin = 0, fuse = 0, yin = 0, lp = 0, flow = 0;
        long long wells = 0;   // 0: no wells, else the wells' version + 1
        bool operator==(const GraphKey &o) const {
            return precision == o.precision && tile_sweeps == o.tile_sweeps && spmv_variant == o.spmv_variant &&
                   sweep_variant == o.sweep_variant && split == o.split && sweep_grid == o.sweep_grid &&
                   spin == o.spin && fuse == o.fuse && yin == o.yin && lp == o.lp && flow == o.flow &&
                   wells == o.wells;
        }
    };
    struct Segment {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        GraphKey key;
    };
    // by iteration parts, plus kRepShift times the number of whole
    // iterations a segment of P_ALL holds beyond one
    std::map<int, Segment> segments;
    void drop_graph() {
        for (auto &kv : segments) {
            if (kv.second.exec) (void)hipGraphExecDestroy(kv.second.exec);
            if (kv.second.graph) (void)hipGraphDestroy(kv.second.graph);
        }
        segments.clear();
    }
    ~rs_ilu0() {
        drop_graph();
        for (hipEvent_t e : {ev_f0, ev_f1, ev_s0, ev_s1, ev_apply})
            if (e) (void)hipEventDestroy(e);
        if (cap_stream) (void)hipStreamDestroy(cap_stream);
        if (pinned) (void)hipHostFree(pinned);
    }
};

static int read_pattern(int32_t n, int32_t nnzb, const int32_t *row_ptr, const int32_t *col_idx, int32_t mem,
                        hipStream_t s, std::vector<int32_t> &rp, std::vector<int32_t> &ci) {
    rp.resize((size_t)n + 1);
    ci.resize((size_t)nnzb);
    if (mem == RS_MEM_DEVICE) {
        HIP_TRY(hipMemcpyAsync(rp.data(), row_ptr, rp.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        if (nnzb) HIP_TRY(hipMemcpyAsync(ci.data(), col_idx, ci.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
    } else {
        std::memcpy(rp.data(), row_ptr, rp.size() * sizeof(int32_t));
        if (nnzb) std::memcpy(ci.data(), col_idx, ci.size() * sizeof(int32_t));
    }
    return RS_OK;
}

extern "C" {

const char *rsolve_last_error(void) { return g_err.c_str(); }

const char *rsolve_status_string(int status) {
    switch (status) {
    case RS_OK: return "ok";
    case RS_NOT_CONVERGED: return "not converged";
    case RS_BREAKDOWN: return "breakdown";
    case RS_PENDING: return "pending";
    case RS_INVALID_ARG: return "invalid argument";
    case RS_UNSUPPORTED_BLOCK_SIZE: return "unsupported block size";
    case RS_BAD_PATTERN: return "bad pattern";
    case RS_MISSING_DIAGONAL: return "missing diagonal block";
    case RS_ZERO_PIVOT: return "zero pivot";
    case RS_NON_FINITE: return "non-finite value";
    case RS_OUT_OF_MEMORY: return "out of memory";
    case RS_HIP_ERROR: return "HIP error";
    case RS_PATTERN_MISMATCH: return "pattern mismatch";
    case RS_NOT_FACTORED: return "not factored";
    default: return "unknown status";
    }
}

int ilu0_analyse_host(int32_t n, const int32_t *row_ptr, const int32_t *col_idx, int32_t ordering, int32_t *perm,
                      int32_t *n_sets, int32_t *bad_row) {
    if (bad_row) *bad_row = -1;
    if (n < 0 || !row_ptr || (n > 0 && !col_idx) || ordering < 0 || ordering > RS_ORDER_RCM_LEVEL_SET)
        return fail(RS_INVALID_ARG, "ilu0_analyse_host: bad arguments");
    int bad = -1;
    const int nnzb = row_ptr[n];
    if (nnzb < 0) return fail(RS_BAD_PATTERN, "ilu0_analyse_host: negative nnzb");
    int st = rs::validate_pattern(n, nnzb, row_ptr, col_idx, &bad);
    if (bad_row) *bad_row = bad;
    if (st != RS_OK) return fail(st, "ilu0_analyse_host: invalid pattern");
    std::vector<int32_t> p, sp;
    const int ns = rs::make_ordering(n, row_ptr, col_idx, ordering, p, sp);
    if (perm && n) std::memcpy(perm, p.data(), sizeof(int32_t) * (size_t)n);
    if (n_sets) *n_sets = ns;
    return RS_OK;
}

int bcsr_create(int32_t n_brows, int32_t nnzb, int32_t block_size, int32_t batch, const int32_t *row_ptr,
                const int32_t *col_idx, const double *vals, int32_t mem, void *stream, bcsr_t *out,
                int32_t *bad_row) {
    if (bad_row) *bad_row = -1;
    if (!out) return fail(RS_INVALID_ARG, "bcsr_create: out is NULL");
    *out = nullptr;
    if (block_size != 3) return fail(RS_UNSUPPORTED_BLOCK_SIZE, "bcsr_create: block size must be 3");
    if (n_brows < 0 || nnzb < 0 || batch < 1 || !row_ptr || (nnzb > 0 && !col_idx) ||
        (mem != RS_MEM_HOST && mem != RS_MEM_DEVICE))
        return fail(RS_INVALID_ARG, "bcsr_create: bad arguments");
    if ((size_t)nnzb * 9 * (size_t)batch > (size_t)1 << 40) return fail(RS_INVALID_ARG, "bcsr_create: too large");
    rs_bcsr *A = new rs_bcsr();
    A->n = n_brows;
    A->nnzb = nnzb;
    A->batch = batch;
    A->spmv_variant = rs::default_sweep_variant(n_brows);   // no dot products: as a sweep
    int st = read_pattern(n_brows, nnzb, row_ptr, col_idx, mem, (hipStream_t)stream, A->h_rowptr, A->h_colidx);
    if (st != RS_OK) { delete A; return st; }
    int bad = -1;
    st = rs::validate_pattern(n_brows, nnzb, A->h_rowptr.data(), A->h_colidx.data(), &bad);
    if (st != RS_OK) {
        if (bad_row) *bad_row = bad;
        delete A;
        return fail(st, "bcsr_create: invalid pattern at row " + std::to_string(bad));
    }
    A->hash = pattern_fingerprint(A->h_rowptr, A->h_colidx);
    hipError_t e;
    if ((e = upload(A->rowptr, A->h_rowptr, (hipStream_t)stream)) != hipSuccess ||
        (e = upload(A->colidx, A->h_colidx, (hipStream_t)stream)) != hipSuccess ||
        (e = A->vals.alloc((size_t)nnzb * 9 * batch * sizeof(double))) != hipSuccess ||
        (e = hipStreamSynchronize((hipStream_t)stream)) != hipSuccess) {
        delete A;
        return fail(e == hipErrorOutOfMemory ? RS_OUT_OF_MEMORY : RS_HIP_ERROR,
                    std::string("bcsr_create: ") + hipGetErrorString(e));
    }
    *out = A;
    if (vals) {
        st = bcsr_set_values(A, vals, 0, batch, mem, stream);
        if (st != RS_OK) {
            delete A;
            *out = nullptr;
            return st;
        }
    }
    return RS_OK;
}

int bcsr_set_values(bcsr_t A, const double *vals, int32_t first_sys, int32_t n_sys, int32_t mem, void *stream) {
    if (!A || !vals || first_sys < 0 || n_sys < 0 || first_sys + n_sys > A->batch)
        return fail(RS_INVALID_ARG, "bcsr_set_values: bad arguments");
    const size_t per = (size_t)A->nnzb * 9;
    if (n_sys == 0 || per == 0) return RS_OK;
    HIP_TRY(hipMemcpyAsync(A->vals.as<double>() + per * first_sys, vals, per * n_sys * sizeof(double),
                           mem == RS_MEM_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                           (hipStream_t)stream));
    if (mem != RS_MEM_DEVICE) HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
    return RS_OK;
}

int bcsr_get_dims(bcsr_t A, int32_t *n_brows, int32_t *nnzb, int32_t *batch) {
    if (!A) return fail(RS_INVALID_ARG, "bcsr_get_dims: NULL handle");
    if (n_brows) *n_brows = A->n;
    if (nnzb) *nnzb = A->nnzb;
    if (batch) *batch = A->batch;
    return RS_OK;
}

int bcsr_set_option(bcsr_t A, int32_t option, int32_t value) {
    if (!A) return fail(RS_INVALID_ARG, "bcsr_set_option: NULL handle");
    if (option == RS_OPT_SPMV_VARIANT && value >= 0 && value < rs::RV_COUNT) {
        A->spmv_variant = value;
        return RS_OK;
    }
    return fail(RS_INVALID_ARG, "bcsr_set_option: unknown option or bad value");
}

int bcsr_set_wells(bcsr_t A, int32_t n_wells, const int32_t *well_ptr, const int32_t *perf_row, const double *B,
                   const double *C, const double *Dinv, int32_t mem, void *stream) {
    if (!A || n_wells < 0 || (mem != RS_MEM_HOST && mem != RS_MEM_DEVICE))
        return fail(RS_INVALID_ARG, "bcsr_set_wells: bad arguments");
    hipStream_t s = (hipStream_t)stream;
    A->wells_version++;
    if (n_wells == 0) {
        A->nw = A->np = 0;
        return RS_OK;
    }
    if (!well_ptr || !perf_row || !B || !C || !Dinv) return fail(RS_INVALID_ARG, "bcsr_set_wells: NULL array");
    if (well_ptr[0] != 0) return fail(RS_INVALID_ARG, "bcsr_set_wells: well_ptr[0] must be 0");
    for (int w = 0; w < n_wells; ++w)
        if (well_ptr[w + 1] < well_ptr[w]) return fail(RS_INVALID_ARG, "bcsr_set_wells: well_ptr decreases");
    const int np = well_ptr[n_wells];
    for (int p = 0; p < np; ++p)
        if (perf_row[p] < 0 || perf_row[p] >= A->n) return fail(RS_INVALID_ARG, "bcsr_set_wells: perforation row out of range");
    A->nw = 0;   // until the copies below are in place
    A->h_well_ptr.assign(well_ptr, well_ptr + n_wells + 1);
    A->h_perf_row.assign(perf_row, perf_row + np);
    A->h_perf_well.resize(np);
    for (int w = 0; w < n_wells; ++w)
        for (int p = well_ptr[w]; p < well_ptr[w + 1]; ++p) A->h_perf_well[p] = w;
    perforation_index(A->n, A->h_perf_row, A->h_row_ptr, A->h_row_perf);
    const size_t Bn = (size_t)A->batch;
    const hipMemcpyKind kind = mem == RS_MEM_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    HIP_TRY(upload(A->w_well_ptr, A->h_well_ptr, s));
    HIP_TRY(upload(A->w_perf_row, A->h_perf_row, s));
    HIP_TRY(upload(A->w_row_ptr, A->h_row_ptr, s));
    HIP_TRY(upload(A->w_row_perf, A->h_row_perf, s));
    HIP_TRY(upload(A->w_perf_well, A->h_perf_well, s));
    HIP_TRY(A->w_B.alloc(std::max<size_t>(Bn * np * 12, 1) * sizeof(double)));
    HIP_TRY(A->w_C.alloc(std::max<size_t>(Bn * np * 12, 1) * sizeof(double)));
    HIP_TRY(A->w_Dinv.alloc(Bn * n_wells * 16 * sizeof(double)));
    HIP_TRY(A->w_t2.alloc(Bn * n_wells * 4 * sizeof(double)));
    if (np) {
        HIP_TRY(hipMemcpyAsync(A->w_B.p, B, Bn * np * 12 * sizeof(double), kind, s));
        HIP_TRY(hipMemcpyAsync(A->w_C.p, C, Bn * np * 12 * sizeof(double), kind, s));
    }
    HIP_TRY(hipMemcpyAsync(A->w_Dinv.p, Dinv, Bn * n_wells * 16 * sizeof(double), kind, s));
    HIP_TRY(hipStreamSynchronize(s));
    A->nw = n_wells;
    A->np = np;
    return RS_OK;
}

int bcsr_destroy(bcsr_t A) {
    delete A;
    return RS_OK;
}

// Stage a caller vector set (nsys systems of 3n doubles) on the device.
static int stage_in(const double *src, int32_t mem, DevBuf &buf, size_t count, hipStream_t s, const double **dev) {
    if (mem == RS_MEM_DEVICE) {
        *dev = src;
        return RS_OK;
    }
    HIP_TRY(buf.alloc(std::max<size_t>(count, 1) * sizeof(double)));
    if (count) HIP_TRY(hipMemcpyAsync(buf.p, src, count * sizeof(double), hipMemcpyHostToDevice, s));
    *dev = buf.as<double>();
    return RS_OK;
}

int bcsr_spmv(bcsr_t A, const double *x, double *y, int32_t first_sys, int32_t n_sys, int32_t mem, void *stream) {
    if (!A || !x || !y || first_sys < 0 || n_sys < 0 || first_sys + n_sys > A->batch)
        return fail(RS_INVALID_ARG, "bcsr_spmv: bad arguments");
    hipStream_t s = (hipStream_t)stream;
    const size_t m = 3 * (size_t)A->n * n_sys;
    DevBuf xb, yb;
    const double *xd = nullptr;
    int st = stage_in(x, mem, xb, m, s, &xd);
    if (st != RS_OK) return st;
    double *yd = y;
    if (mem != RS_MEM_DEVICE) {
        HIP_TRY(yb.alloc(std::max<size_t>(m, 1) * sizeof(double)));
        yd = yb.as<double>();
    }
    const size_t per = (size_t)A->nnzb * 9;
    rs::launch_spmv(A->n, A->rowptr.as<int32_t>(), A->colidx.as<int32_t>(), A->vals.as<double>() + per * first_sys,
                    per, xd, yd, 3 * (size_t)A->n, n_sys, A->spmv_variant, A->wells(first_sys), s);
    HIP_TRY(hipGetLastError());
    if (mem != RS_MEM_DEVICE) {
        if (m) HIP_TRY(hipMemcpyAsync(y, yd, m * sizeof(double), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
    }
    return RS_OK;
}

static int build_analysis(const rs_bcsr *A, int32_t ordering, const int32_t *part, std::shared_ptr<Analysis> &out) {
    auto an = std::make_shared<Analysis>();
    an->hash = A->hash;
    rs::build_schedule(A->n, A->nnzb, A->h_rowptr.data(), A->h_colidx.data(), ordering, an->sch, rs::kFlowRows,
                       rs::kApplyRows, rs::kApplyRowsSmall, part);
    const rs::Schedule &S = an->sch;
    for (int q = 0; q < S.n; ++q)
        if (S.lptr[q + 1] > S.lptr[q]) an->u_kept += S.uptr[S.l2u[q] + 1] - S.uptr[S.l2u[q]];
    hipError_t e = hipSuccess;
    struct Up { DevBuf *b; const std::vector<int32_t> *v; } ups[] = {
        {&an->perm, &S.perm}, {&an->prow, &S.prow}, {&an->pcol, &S.pcol}, {&an->psrc, &S.psrc},
        {&an->lrows, &S.lrows}, {&an->lptr, &S.lptr}, {&an->lcol, &S.lcol}, {&an->lsrc, &S.lsrc},
        {&an->ldq, &S.ldq}, {&an->l2u, &S.l2u}, {&an->upd_ptr, &S.upd_ptr}, {&an->upd, &S.upd},
        {&an->urows, &S.urows}, {&an->uptr, &S.uptr}, {&an->ucol, &S.ucol}, {&an->usrc, &S.usrc},
        {&an->dsrc, &S.dsrc}, {&an->lsrc_a, &S.lsrc_a}, {&an->usrc_a, &S.usrc_a}, {&an->dsrc_a, &S.dsrc_a},
        {&an->rest_dst, &S.rest_dst}, {&an->rest_src, &S.rest_src}, {&an->lt_start, &S.ltiles},
        {&an->ut_start, &S.utiles}, {&an->la_start, &S.tiles_large.lt}, {&an->ua_start, &S.tiles_large.ut},
        {&an->ls_start, &S.tiles_small.lt}, {&an->us_start, &S.tiles_small.ut}};
    // uploads on a private stream, complete before the handle is returned,
    // so that any stream may use the analysis
    hipStream_t us = nullptr;
    e = hipStreamCreateWithFlags(&us, hipStreamNonBlocking);
    if (e == hipSuccess) {
        for (auto &u : ups)
            if ((e = upload(*u.b, *u.v, us)) != hipSuccess) break;
        const hipError_t e2 = hipStreamSynchronize(us);
        if (e == hipSuccess) e = e2;
        (void)hipStreamDestroy(us);
    }
    if (e != hipSuccess)
        return fail(e == hipErrorOutOfMemory ? RS_OUT_OF_MEMORY : RS_HIP_ERROR,
                    std::string("ilu0_analyse: ") + hipGetErrorString(e));
    DevSchedule &d = an->dev;
    d.n = S.n; d.nnzb = S.nnzb; d.nL = S.nL; d.nU = S.nU;
    d.perm = an->perm.as<int32_t>(); d.prow = an->prow.as<int32_t>(); d.pcol = an->pcol.as<int32_t>();
    d.psrc = an->psrc.as<int32_t>(); d.lrows = an->lrows.as<int32_t>(); d.lptr = an->lptr.as<int32_t>();
    d.lcol = an->lcol.as<int32_t>(); d.lsrc = an->lsrc.as<int32_t>(); d.ldq = an->ldq.as<int32_t>();
    d.l2u = an->l2u.as<int32_t>(); d.upd_ptr = an->upd_ptr.as<int32_t>(); d.upd = an->upd.as<int32_t>();
    d.urows = an->urows.as<int32_t>(); d.uptr = an->uptr.as<int32_t>(); d.ucol = an->ucol.as<int32_t>();
    d.usrc = an->usrc.as<int32_t>(); d.dsrc = an->dsrc.as<int32_t>();
    d.lsrc_a = an->lsrc_a.as<int32_t>(); d.usrc_a = an->usrc_a.as<int32_t>(); d.dsrc_a = an->dsrc_a.as<int32_t>();
    d.nrest = (int)S.rest_dst.size();
    d.rest_dst = an->rest_dst.as<int32_t>(); d.rest_src = an->rest_src.as<int32_t>();
    d.fuse_n0 = S.fuse_n0; d.fuse_q0 = S.fuse_q0; d.y_last = S.y_last;
    d.nlt = (int)S.ltiles.size() - 1; d.nut = (int)S.utiles.size() - 1;
    d.lt_start = an->lt_start.as<int32_t>(); d.ut_start = an->ut_start.as<int32_t>();
    auto tiles = [](const rs::Schedule::ApplyTiles &t, const DevBuf &lt, const DevBuf &ut) {
        return DevSchedule::ApplyTiles{lt.as<int32_t>(), ut.as<int32_t>(), (int)t.lt.size() - 1, (int)t.ut.size() - 1,
                                       t.uf0, t.nf};
    };
    d.tiles_large = tiles(S.tiles_large, an->la_start, an->ua_start);
    d.tiles_small = tiles(S.tiles_small, an->ls_start, an->us_start);
    out = std::move(an);
    return RS_OK;
}

static rs_ilu0 *new_ilu0(const rs_bcsr *A, std::shared_ptr<const Analysis> an) {
    rs_ilu0 *M = new rs_ilu0();
    M->n = A->n;
    M->nnzb = A->nnzb;
    M->batch = A->batch;
    M->hash = A->hash;
    M->spmv_variant = rs::default_spmv_variant(M->n, M->batch);
    M->sweep_variant = rs::default_sweep_variant(M->n);
    // many thin levels (natural order, level sets): one launch per sweep;
    // few wide colours or levels (colouring, RCM then level sets): one
    // launch per colour or level
    M->tile_sweeps = an->sch.ordering == RS_ORDER_NATURAL || an->sch.ordering == RS_ORDER_LEVEL_SET;
    M->an = std::move(an);
    return M;
}

int ilu0_analyse(bcsr_t A, int32_t ordering, ilu0_t *out) {
    if (!A || !out || ordering < 0 || ordering > RS_ORDER_RCM_LEVEL_SET)
        return fail(RS_INVALID_ARG, "ilu0_analyse: bad arguments");
    *out = nullptr;
    std::shared_ptr<Analysis> an;
    const int st = build_analysis(A, ordering, nullptr, an);
    if (st != RS_OK) return st;
    *out = new_ilu0(A, std::move(an));
    return RS_OK;
}

int ilu0_analyse_jacobi(bcsr_t A, int32_t ordering, const int32_t *part, ilu0_t *out) {
    if (!A || !out || !part || ordering < 0 || ordering > RS_ORDER_RCM_LEVEL_SET)
        return fail(RS_INVALID_ARG, "ilu0_analyse_jacobi: bad arguments");
    *out = nullptr;
    std::shared_ptr<Analysis> an;
    const int st = build_analysis(A, ordering, part, an);
    if (st != RS_OK) return st;
    *out = new_ilu0(A, std::move(an));
    return RS_OK;
}

int bcsr_partition(int32_t n_brows, int32_t nnzb, const int32_t *row_ptr, const int32_t *col_idx,
                   const double *weights, int32_t n_parts, int32_t *part) {
    if (n_brows < 0 || nnzb < 0 || !row_ptr || (nnzb > 0 && !col_idx) || n_parts < 1 || (n_brows > 0 && !part))
        return fail(RS_INVALID_ARG, "bcsr_partition: bad arguments");
    int bad = -1;
    const int st = rs::validate_pattern(n_brows, nnzb, row_ptr, col_idx, &bad);
    if (st != RS_OK) return fail(st, "bcsr_partition: invalid pattern at row " + std::to_string(bad));
    rs::partition_rows(n_brows, row_ptr, col_idx, weights, n_parts, part);
    return RS_OK;
}

int ilu0_analyse_shared(bcsr_t A, ilu0_t like, ilu0_t *out) {
    if (!A || !like || !out) return fail(RS_INVALID_ARG, "ilu0_analyse_shared: bad arguments");
    *out = nullptr;
    if (A->n != like->n || A->nnzb != like->nnzb || A->hash != like->an->hash)
        return fail(RS_PATTERN_MISMATCH, "ilu0_analyse_shared: A's pattern differs from the analysed one");
    *out = new_ilu0(A, like->an);
    return RS_OK;
}

int ilu0_get_schedule(ilu0_t M, int32_t *perm, int32_t *n_sets, int32_t *set_ptr) {
    if (!M) return fail(RS_INVALID_ARG, "ilu0_get_schedule: NULL handle");
    if (perm && M->n) std::memcpy(perm, M->an->sch.perm.data(), sizeof(int32_t) * (size_t)M->n);
    if (n_sets) *n_sets = M->an->sch.n_sets;
    if (set_ptr) std::memcpy(set_ptr, M->an->sch.set_ptr.data(), sizeof(int32_t) * M->an->sch.set_ptr.size());
    return RS_OK;
}

int ilu0_get_sweep_levels(ilu0_t M, int32_t *n_lower, int32_t *n_upper) {
    if (!M) return fail(RS_INVALID_ARG, "ilu0_get_sweep_levels: NULL handle");
    if (n_lower) *n_lower = M->an->sch.nl_levels;
    if (n_upper) *n_upper = M->an->sch.nu_levels;
    return RS_OK;
}

int ilu0_set_option(ilu0_t M, int32_t option, int32_t value) {
    if (!M) return fail(RS_INVALID_ARG, "ilu0_set_option: NULL handle");
    switch (option) {
    case RS_OPT_SWEEP_TILES:
        if (value != 0 && value != 1) break;
        M->tile_sweeps = value != 0;
        return RS_OK;
    case RS_OPT_SWEEP_GRID:
        if (value < 1) break;
        M->sweep_grid = value;
        return RS_OK;
    case RS_OPT_POLL_CHUNK:
        if (value < 1) break;
        M->chunk = value;
        return RS_OK;
    case RS_OPT_USE_GRAPH:
        if (value != 0 && value != 1) break;
        M->use_graph = value != 0;
        return RS_OK;
    case RS_OPT_PREDICT_POLL:
        if (value != 0 && value != 1) break;
        M->predict = value != 0;
        return RS_OK;
    case RS_OPT_SPMV_VARIANT:
        if (value < 0 || value >= rs::RV_COUNT) break;
        M->spmv_variant = value;
        return RS_OK;
    case RS_OPT_REDUCE_SPLIT:
        if (value < 0 || value > 2) break;
        M->reduce_split = value;
        return RS_OK;
    case RS_OPT_SWEEP_VARIANT:
        if (value < 0 || value >= rs::RV_COUNT) break;
        M->sweep_variant = value;
        return RS_OK;
    case RS_OPT_SPIN_LIMIT:
        if (value < 0) break;
        M->spin_limit = value;
        return RS_OK;
    case RS_OPT_FUSE_SPMV:
        if (value != 0 && value != 1) break;
        M->fuse_spmv = value != 0;
        return RS_OK;
    case RS_OPT_Y_INPUT:
        if (value != 0 && value != 1) break;
        M->y_input = value != 0;
        return RS_OK;
    case RS_OPT_FACTOR_ASYNC:
        if (value != 0 && value != 1) break;
        M->factor_async = value != 0;
        return RS_OK;
    case RS_OPT_LOWER_PARTS:
        if (value != 0 && value != 1) break;
        M->lower_parts = value != 0;
        return RS_OK;
    default:
        break;
    }
    return fail(RS_INVALID_ARG, "ilu0_set_option: unknown option or bad value");
}

int ilu0_get_option(ilu0_t M, int32_t option, int32_t *value) {
    if (!M || !value) return fail(RS_INVALID_ARG, "ilu0_get_option: bad arguments");
    switch (option) {
    case RS_OPT_SWEEP_TILES: *value = M->tile_sweeps ? 1 : 0; return RS_OK;
    case RS_OPT_SWEEP_GRID: *value = M->sweep_grid; return RS_OK;
    case RS_OPT_POLL_CHUNK: *value = M->chunk; return RS_OK;
    case RS_OPT_USE_GRAPH: *value = M->use_graph ? 1 : 0; return RS_OK;
    case RS_OPT_PREDICT_POLL: *value = M->predict ? 1 : 0; return RS_OK;
    case RS_OPT_SPMV_VARIANT: *value = M->spmv_variant; return RS_OK;
    case RS_OPT_SWEEP_VARIANT: *value = M->sweep_variant; return RS_OK;
    case RS_OPT_REDUCE_SPLIT: *value = M->reduce_split; return RS_OK;
    case RS_OPT_SPIN_LIMIT: *value = M->spin_limit; return RS_OK;
    case RS_OPT_FUSE_SPMV: *value = M->fuse_spmv ? 1 : 0; return RS_OK;
    case RS_OPT_FUSED_ROWS: *value = M->an->sch.fuse_n0; return RS_OK;
    case RS_OPT_Y_INPUT: *value = M->y_input ? 1 : 0; return RS_OK;
    case RS_OPT_Y_INPUT_PATTERN: *value = M->an->sch.y_in; return RS_OK;
    case RS_OPT_FACTOR_ASYNC: *value = M->factor_async ? 1 : 0; return RS_OK;
    case RS_OPT_LOWER_PARTS: *value = M->lower_parts ? 1 : 0; return RS_OK;
    default: return fail(RS_INVALID_ARG, "ilu0_get_option: unknown option");
    }
}

// U blocks of the fused rows, when the factorisation did not store them,
// for a consumer that reads U: copied from A' (rounded to FP32 with FP32
// factors) on `s`, once per factorisation.
static int ensure_u(ilu0_t M, hipStream_t s) {
    if (!M->u_missing) return RS_OK;
    const rs::Schedule &S = M->an->sch;
    const int f0 = S.uptr[S.fuse_q0], f1 = S.uptr[S.fuse_q0 + S.fuse_n0];
    if (M->precision == RS_PREC_FP32_FACTORS)
        rs::launch_fill_u<float>(M->an->dev, M->pvals.as<double>(), (size_t)M->nnzb * 9, M->Uf.as<float>(),
                                 (size_t)S.nU * 9, f0, f1, M->batch, s);
    else
        rs::launch_fill_u<double>(M->an->dev, M->pvals.as<double>(), (size_t)M->nnzb * 9, M->U.as<double>(),
                                  (size_t)S.nU * 9, f0, f1, M->batch, s);
    HIP_TRY(hipGetLastError());
    M->u_missing = false;
    return RS_OK;
}

// Whether the coming launches read U of the fused rows: single-launch
// sweeps always, and with FP32 factors every upper launch outside BiCGStab's
// fused iteration (per-level upper launches of FP64 factors read A').
static bool reads_u(const rs_ilu0 *M, bool fused) {
    return M->tile_sweeps || (M->precision == RS_PREC_FP32_FACTORS && !fused);
}

static void factor_message(int status) {
    g_err = status == RS_ZERO_PIVOT ? "ilu0_factor: singular pivot block"
                                    : "ilu0_factor: a row's dependency wait exceeded its limit";
}

// The result of the handle's last factorisation, which has completed and
// whose first singular pivots (new numbering) are in bad_host: device time,
// per-system bad rows (original numbering, -1 when none), status.
static int factor_result(ilu0_t M, int32_t *bad_row) {
    const size_t B = (size_t)M->batch;
    float ms = 0.f;
    M->factor_ms = hipEventElapsedTime(&ms, M->ev_f0, M->ev_f1) == hipSuccess ? ms : 0.0;
    int worst = RS_OK;
    M->bad_orig.assign(B, -1);
    bool gave_up = false;
    for (size_t i = 0; i < B; ++i) {
        const int32_t b = M->bad_host[i];
        if (b == rs::kBadWait) gave_up = true;
        const int32_t orig = (b >= 0 && b < M->n) ? M->an->sch.perm[b] : -1;
        M->bad_orig[i] = orig;
        if (orig >= 0) worst = RS_ZERO_PIVOT;
    }
    if (gave_up) worst = RS_HIP_ERROR;
    if (bad_row) std::copy(M->bad_orig.begin(), M->bad_orig.end(), bad_row);
    M->factor_status = worst;
    M->factor_pending = false;
    if (worst != RS_OK) factor_message(worst);
    return worst;
}

// Device time of the last factorisation for a solve's info: a queued one
// has completed once the solve that follows it on the same stream has.
static double factor_time(ilu0_t M) {
    if (!M->factor_pending) return M->factor_ms;
    float ms = 0.f;
    return hipEventElapsedTime(&ms, M->ev_f0, M->ev_f1) == hipSuccess ? ms : 0.0;
}

static bool capturing(hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
    return cap != hipStreamCaptureStatusNone;
}

// Order `s` after the handle's last queued application (ilu0_apply), whatever
// stream that was on.  A stream being captured may not depend on work outside
// its capture: there the host waits for the application (in the relaxed mode,
// since the wait is none of the capture's business).  That wait would
// invalidate a capture of the application's own stream; what such a capture
// records comes after the application by the order of the caller's launch.
static int after_apply(ilu0_t M, hipStream_t s) {
    if (!M->apply_queued) return RS_OK;
    if (!capturing(s)) {
        HIP_TRY(hipStreamWaitEvent(s, M->ev_apply, 0));
        return RS_OK;
    }
    if (capturing(M->apply_stream)) return RS_OK;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    HIP_TRY(hipThreadExchangeStreamCaptureMode(&mode));
    const hipError_t e = hipEventSynchronize(M->ev_apply);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    HIP_TRY(e);
    M->apply_queued = false;
    return RS_OK;
}

// The calls that wait for their stream end with an error in a capture; they
// end before any work, so that nothing the handle notes as done (y marked) is
// only recorded.
static int refuse_capture(hipStream_t s, const char *call) {
    if (!capturing(s)) return RS_OK;
    return fail(RS_HIP_ERROR, std::string(call) + ": the stream is being captured");
}

static int check_pair(ilu0_t M, bcsr_t A) {
    if (!M || !A) return fail(RS_INVALID_ARG, "NULL handle");
    if (M->hash != A->hash || M->n != A->n || M->nnzb != A->nnzb)
        return fail(RS_PATTERN_MISMATCH, "ilu0 handle analysed for another pattern");
    if (M->batch != A->batch) return fail(RS_PATTERN_MISMATCH, "batch size differs from the analysed matrix");
    return RS_OK;
}

static int ensure_pinned(ilu0_t M) {
    if (M->pinned) return RS_OK;
    const size_t B = (size_t)M->batch;
    auto after = [](size_t at, size_t bytes) { return (at + bytes + 255) / 256 * 256; };
    const size_t at_state = after(0, 2 * sizeof(rs::SweepCtr)), at_bad = after(at_state, B * sizeof(SysState));
    HIP_TRY(hipHostMalloc(&M->pinned, at_bad + B * sizeof(int32_t), hipHostMallocDefault));
    unsigned char *p = (unsigned char *)M->pinned;
    M->h_ctr = (rs::SweepCtr *)p;
    M->h_state = (SysState *)(p + at_state);
    M->bad_host = (int32_t *)(p + at_bad);
    return RS_OK;
}

constexpr int kFlowFactorRows = 12000;   // see ilu0_factor

int ilu0_factor(ilu0_t M, bcsr_t A, int32_t precision, void *stream, int32_t *bad_row) {
    int st = check_pair(M, A);
    if (st != RS_OK) return st;
    if (precision != RS_PREC_FP64 && precision != RS_PREC_FP32_FACTORS)
        return fail(RS_INVALID_ARG, "ilu0_factor: unknown precision");
    hipStream_t s = (hipStream_t)stream;
    if ((st = after_apply(M, s)) != RS_OK) return st;
    const rs::Schedule &S = M->an->sch;
    const size_t B = (size_t)M->batch;
    HIP_TRY(M->pvals.alloc(B * M->nnzb * 9 * sizeof(double)));
    HIP_TRY(M->L.alloc(B * S.nL * 9 * sizeof(double)));
    HIP_TRY(M->U.alloc(B * S.nU * 9 * sizeof(double)));
    HIP_TRY(M->Dinv.alloc(B * M->n * 9 * sizeof(double)));
    HIP_TRY(M->bad.alloc(B * sizeof(int32_t)));
    if (precision == RS_PREC_FP32_FACTORS) {
        HIP_TRY(M->Lf.alloc(B * S.nL * 9 * sizeof(float)));
        HIP_TRY(M->Uf.alloc(B * S.nU * 9 * sizeof(float)));
        HIP_TRY(M->Dinvf.alloc(B * M->n * 9 * sizeof(float)));
    }
    M->factored = false;
    if ((st = ensure_pinned(M)) != RS_OK) return st;
    if (!M->ev_f0) HIP_TRY(hipEventCreate(&M->ev_f0));
    if (!M->ev_f1) HIP_TRY(hipEventCreate(&M->ev_f1));
    HIP_TRY(hipEventRecord(M->ev_f0, s));
    const size_t per = (size_t)M->nnzb * 9;
    // One launch over all levels while a level holds few rows (of all
    // systems): a launch per level costs 11-12 us whatever its size, a level
    // inside the one launch 1.5-4 us, but that launch keeps one workgroup a
    // CU, so wide levels leave the memory idle in it.  33 levels of 3 400
    // rows (Block-Jacobi, 113k cells) take 135 instead of 414 us, four of
    // 24 000 (96k cells, colouring) 94 instead of 84.
    const bool flow = (double)M->n * M->batch <= (double)kFlowFactorRows * S.nl_levels && S.nl_levels > 2;
    if (flow) HIP_TRY(M->fctr.alloc(sizeof(rs::SweepCtr)));
    else HIP_TRY(hipMemsetAsync(M->bad.p, 0x7f, B * sizeof(int32_t), s));
    {
        // algorithmic bytes of the method: every block of the
        // preconditioner's matrix read, updated in place and written once
        // (148 per block with its index); Block-Jacobi also copies the
        // dropped blocks into A' (144 each)
        const double bytes = 148.0 * S.nnz_m + 144.0 * (double)S.rest_dst.size();
        ProfScope ps(PC_FACTOR, s, B * bytes);
        const DevSchedule &d = M->an->dev;
        const bool f32 = precision == RS_PREC_FP32_FACTORS;
        // the U of the fused rows is their rows of A', which their upper
        // launches read instead (filled in later for a consumer of U)
        const bool skip_u0 = S.fuse_n0 > 0;
        // a first level made of those rows is a copy and a pivot inversion
        const bool first = S.fuse_n0 > 0 && S.nl_levels > 0 && S.lset[1] == S.fuse_n0 && S.lconsec[0] &&
                           S.rest_dst.empty();
        if (flow)
            rs::launch_factor_flow(d, A->vals.as<double>(), per, M->pvals.as<double>(), M->L.as<double>(),
                                   M->U.as<double>(), M->Dinv.as<double>(), f32 ? M->Lf.as<float>() : nullptr,
                                   f32 ? M->Uf.as<float>() : nullptr, f32 ? M->Dinvf.as<float>() : nullptr,
                                   M->bad.as<int32_t>(), skip_u0,
                                   std::find(S.lnarrow.begin(), S.lnarrow.end(), 0) == S.lnarrow.end(), S.nl_levels,
                                   M->spin_limit, M->fctr.as<rs::SweepCtr>(), M->batch, s);
        else
            rs::launch_gather_pairs(A->vals.as<double>(), per, M->pvals.as<double>(), per, d.rest_dst, d.rest_src,
                                    d.nrest, M->batch, s);
        for (int l = 0; !flow && l < S.nl_levels; ++l) {
            if (l == 0 && first) {
                rs::launch_factor_first(d, A->vals.as<double>(), per, M->pvals.as<double>(), M->Dinv.as<double>(),
                                        f32 ? M->Dinvf.as<float>() : nullptr, M->bad.as<int32_t>(), M->batch, s);
                continue;
            }
            rs::launch_factor_level(d, A->vals.as<double>(), per, M->pvals.as<double>(), M->L.as<double>(),
                                    M->U.as<double>(), M->Dinv.as<double>(), f32 ? M->Lf.as<float>() : nullptr,
                                    f32 ? M->Uf.as<float>() : nullptr, f32 ? M->Dinvf.as<float>() : nullptr,
                                    M->bad.as<int32_t>(), S.lset[l], S.lset[l + 1],
                                    S.lconsec[l] && S.rest_dst.empty(), skip_u0, l == S.nl_levels - 1,
                                    S.lnarrow[l] != 0, M->batch, s);
        }
        M->u_missing = skip_u0;
    }
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipEventRecord(M->ev_f1, s));
    M->precision = precision;
    M->factored = true;
    M->factor_pending = true;
    if (M->factor_async) return RS_OK;
    HIP_TRY(hipMemcpyAsync(M->bad_host, M->bad.p, B * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    M->apply_queued = false;   // `s` came after it
    return factor_result(M, bad_row);
}

int ilu0_factor_status(ilu0_t M, int32_t *bad_row) {
    if (!M) return fail(RS_INVALID_ARG, "ilu0_factor_status: NULL handle");
    if (!M->factored) return fail(RS_NOT_FACTORED, "ilu0_factor_status: not factored");
    if (M->factor_pending) {
        HIP_TRY(hipEventSynchronize(M->ev_f1));
        HIP_TRY(hipMemcpy(M->bad_host, M->bad.p, M->batch * sizeof(int32_t), hipMemcpyDeviceToHost));
        return factor_result(M, bad_row);
    }
    if (bad_row) std::copy(M->bad_orig.begin(), M->bad_orig.end(), bad_row);
    if (M->factor_status != RS_OK) factor_message(M->factor_status);
    return M->factor_status;
}

int ilu0_get_factors(ilu0_t M, int32_t sys, double *lu, double *dinv) {
    if (!M || sys < 0 || sys >= M->batch) return fail(RS_INVALID_ARG, "ilu0_get_factors: bad arguments");
    if (!M->factored) return fail(RS_NOT_FACTORED, "ilu0_get_factors: not factored");
    HIP_TRY(hipDeviceSynchronize());   // the factorisation may still run on any stream
    int st = ensure_u(M, nullptr);
    if (st != RS_OK) return st;
    HIP_TRY(hipDeviceSynchronize());
    const rs::Schedule &S = M->an->sch;
    if (lu) std::memset(lu, 0, sizeof(double) * 9 * (size_t)M->nnzb);   // diagonal, blocks outside a Jacobi matrix
    std::vector<double> L((size_t)S.nL * 9), U((size_t)S.nU * 9), D((size_t)M->n * 9);
    if (M->precision == RS_PREC_FP32_FACTORS) {
        std::vector<float> Lf(L.size()), Uf(U.size()), Df(D.size());
        if (!Lf.empty()) HIP_TRY(hipMemcpy(Lf.data(), M->Lf.as<float>() + (size_t)sys * Lf.size(), Lf.size() * 4, hipMemcpyDeviceToHost));
        if (!Uf.empty()) HIP_TRY(hipMemcpy(Uf.data(), M->Uf.as<float>() + (size_t)sys * Uf.size(), Uf.size() * 4, hipMemcpyDeviceToHost));
        if (!Df.empty()) HIP_TRY(hipMemcpy(Df.data(), M->Dinvf.as<float>() + (size_t)sys * Df.size(), Df.size() * 4, hipMemcpyDeviceToHost));
        std::copy(Lf.begin(), Lf.end(), L.begin());
        std::copy(Uf.begin(), Uf.end(), U.begin());
        std::copy(Df.begin(), Df.end(), D.begin());
    } else {
        if (!L.empty()) HIP_TRY(hipMemcpy(L.data(), M->L.as<double>() + (size_t)sys * L.size(), L.size() * 8, hipMemcpyDeviceToHost));
        if (!U.empty()) HIP_TRY(hipMemcpy(U.data(), M->U.as<double>() + (size_t)sys * U.size(), U.size() * 8, hipMemcpyDeviceToHost));
        if (!D.empty()) HIP_TRY(hipMemcpy(D.data(), M->Dinv.as<double>() + (size_t)sys * D.size(), D.size() * 8, hipMemcpyDeviceToHost));
    }
    if (lu) {
        for (int e = 0; e < S.nL; ++e) std::memcpy(lu + (size_t)S.lsrc[e] * 9, &L[(size_t)e * 9], 72);
        for (int f = 0; f < S.nU; ++f) std::memcpy(lu + (size_t)S.usrc[f] * 9, &U[(size_t)f * 9], 72);
    }
    if (dinv)
        for (int q = 0; q < M->n; ++q) std::memcpy(dinv + (size_t)S.urows[q] * 9, &D[(size_t)q * 9], 72);
    return RS_OK;
}

// The matrix's wells in the new numbering (rebuilt when A or its wells
// change); ordered on `s`.
static int ensure_wells(ilu0_t M, const rs_bcsr *A, hipStream_t s) {
    if (A->nw == 0) {
        M->wdev = rs::WellsDev{};
        M->wells_of = A;
        M->wells_version = A->wells_version;
        return RS_OK;
    }
    if (M->wells_of != A || M->wells_version != A->wells_version) {
        const std::vector<int32_t> &iperm = M->an->sch.iperm;
        M->h_wperf_x.resize(A->np);
        for (int p = 0; p < A->np; ++p) M->h_wperf_x[p] = iperm[A->h_perf_row[p]];
        perforation_index(M->n, M->h_wperf_x, M->h_wrow_ptr, M->h_wrow_perf);
        HIP_TRY(upload(M->wperf_x, M->h_wperf_x, s));
        HIP_TRY(upload(M->wrow_ptr, M->h_wrow_ptr, s));
        HIP_TRY(upload(M->wrow_perf, M->h_wrow_perf, s));
        M->h_wfix.clear();
        for (int i = 0; i < M->an->sch.fuse_n0; ++i)
            if (M->h_wrow_ptr[i + 1] > M->h_wrow_ptr[i]) M->h_wfix.push_back(i);
        HIP_TRY(upload(M->wfix, M->h_wfix, s));
        HIP_TRY(M->wt2.alloc((size_t)M->batch * A->nw * 4 * sizeof(double)));
        M->wells_of = A;
        M->wells_version = A->wells_version;
    }
    rs::WellsDev w = A->wells();
    w.perf_x = M->wperf_x.as<int32_t>();
    w.row_ptr = M->wrow_ptr.as<int32_t>();
    w.row_perf = M->wrow_perf.as<int32_t>();
    w.t2 = M->wt2.as<double>();
    w.nfix = (int)M->h_wfix.size();
    w.fix_row = M->wfix.as<int32_t>();
    M->wdev = w;
    return RS_OK;
}

// Allocate (first call) and bind the solve workspace; initialisation is
// ordered on the caller's stream `s`.
static int ensure_workspace(ilu0_t M, hipStream_t s) {
    const int pin = ensure_pinned(M);
    if (pin != RS_OK) return pin;
    const size_t B = (size_t)M->batch, vs = rs::vec_stride(M->n);
    const size_t vec = std::max<size_t>(B * vs, 1);
    if (!M->work.p) {
        HIP_TRY(M->work.alloc(9 * vec * sizeof(double)));
        HIP_TRY(hipMemsetAsync(M->work.p, 0, 9 * vec * sizeof(double), s));  // padding stays zero
    }
    HIP_TRY(M->ywork.alloc(vec * sizeof(double)));
    const int max_blocks = std::max(rs::row_blocks(std::max(M->n, 1), 1), rs::kVecMaxBlocks);
    const size_t pstride = rs::part_stride_for(max_blocks), tstride = rs::ticket_stride_for(max_blocks);
    if (!M->part.p || M->k.part_stride != pstride) HIP_TRY(M->part.alloc(B * pstride * sizeof(double)));
    const size_t sstride = rs::part_stride_for(rs::row_blocks(std::max(M->n, 1), 1));
    if (!M->spart.p) HIP_TRY(M->spart.alloc(B * sstride * sizeof(double)));
    const size_t fstride = rs::part_stride_for(rs::fuse_blocks(M->an->sch.fuse_n0, 1));
    if (!M->fpart.p) HIP_TRY(M->fpart.alloc(B * fstride * sizeof(double)));
    if (!M->tickets.p) {
        HIP_TRY(M->tickets.alloc(B * tstride * sizeof(uint32_t)));
        HIP_TRY(hipMemsetAsync(M->tickets.p, 0, B * tstride * sizeof(uint32_t), s));
    }
    if (!M->state.p) {
        HIP_TRY(M->state.alloc(B * sizeof(SysState)));
        HIP_TRY(hipMemsetAsync(M->state.p, 0, B * sizeof(SysState), s));
    }
    if (!M->ctrs.p) {
        HIP_TRY(M->ctrs.alloc(2 * sizeof(rs::SweepCtr)));
        HIP_TRY(hipMemsetAsync(M->ctrs.p, 0, 2 * sizeof(rs::SweepCtr), s));
    }
    if (!M->vpart.p) {
        HIP_TRY(M->vpart.alloc(M->vpart_bytes()));
        rs::launch_flow_mark(M->vpart.p, M->vpart_bytes(), s);
        HIP_TRY(hipGetLastError());
    }
    double *w = M->work.as<double>();
    Krylov &k = M->k;
    k.vpart = M->vpart.as<double>();
    k.vpart_stride = M->vpart_stride();
    k.r = w; k.rhat = w + vec; k.p = w + 2 * vec; k.v = w + 3 * vec; k.phat = w + 4 * vec;
    k.s = w + 5 * vec; k.shat = w + 6 * vec; k.t = w + 7 * vec; k.x = w + 8 * vec;
    k.vstride = vs;
    k.y = M->ywork.p;
    k.y2 = M->ywork2.p;
    k.ftickets = M->ftickets.as<uint32_t>();
    k.fticket_stride = (uint32_t)rs::ticket_stride_for(rs::fuse_blocks(M->an->sch.fuse_n0, 1));
    k.part = M->part.as<double>();
    k.part_stride = pstride;
    k.tickets = M->tickets.as<uint32_t>();
    k.ticket_stride = tstride;
    k.spart = M->spart.as<double>();
    k.spart_stride = sstride;
    k.fpart = M->fpart.as<double>();
    k.fpart_stride = fstride;
    k.lp = M->lpwork.p ? M->lpwork.as<double>() : nullptr;
    k.st = M->state.as<SysState>();
    k.spin = M->spin_limit;
    k.lctr = M->ctrs.as<rs::SweepCtr>();
    k.uctr = k.lctr + 1;
    // single-launch sweeps find y marked and leave it so; per-level sweeps
    // store y over the marks
    if (!M->tile_sweeps) M->y_marked = false;
    else if (!M->y_marked) {
        rs::launch_flow_mark(M->ywork.p, vec * sizeof(double), s);
        HIP_TRY(hipGetLastError());
        M->y_marked = true;
    }
    return RS_OK;
}

// After a wait gave up: clear the sweep counters and have y marked again, once
// the stream has drained.
static int sweep_reset(ilu0_t M, hipStream_t s) {
    HIP_TRY(hipMemsetAsync(M->ctrs.p, 0, 2 * sizeof(rs::SweepCtr), s));
    M->y_marked = false;
    HIP_TRY(hipStreamSynchronize(s));
    return fail(RS_HIP_ERROR, "sweep dependency wait exceeded its limit");
}

// After a solve (its states and, with `ctrs`, the sweep counters are on the
// host): RS_HIP_ERROR when one of its waits gave up, with everything a late
// store of that launch may have touched set anew.
static int solve_waits(ilu0_t M, bool ctrs, hipStream_t s) {
    int st = RS_OK;
    if (ctrs && (M->h_ctr[0].error || M->h_ctr[1].error)) st = sweep_reset(M, s);
    bool gave_up = false;
    for (int i = 0; i < M->batch; ++i) gave_up = gave_up || M->h_state[i].gave_up;
    if (!gave_up) return st;
    HIP_TRY(hipMemsetAsync(M->state.p, 0, (size_t)M->batch * sizeof(SysState), s));
    rs::launch_flow_mark(M->vpart.p, M->vpart_bytes(), s);
    if (M->gm_vpart.p) rs::launch_flow_mark(M->gm_vpart.p, M->gm_vpart_bytes(), s);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(s));
    return st != RS_OK ? st : fail(RS_HIP_ERROR, "reduction wait exceeded its limit");
}

// Events bracketing a solve call on its stream (created on first use); the
// start is recorded here.
static int solve_events(ilu0_t M, hipStream_t s) {
    if (!M->ev_s0) HIP_TRY(hipEventCreate(&M->ev_s0));
    if (!M->ev_s1) HIP_TRY(hipEventCreate(&M->ev_s1));
    HIP_TRY(hipEventRecord(M->ev_s0, s));
    return RS_OK;
}

static double elapsed_ms(hipEvent_t a, hipEvent_t b) {
    float ms = 0.f;
    return hipEventElapsedTime(&ms, a, b) == hipSuccess ? ms : 0.0;
}

// Largest number of iterations (GMRES: steps) a solve queues before its
// first poll when predicting from the previous solve.
constexpr int kPredictMax = 50;

// Non-zero when a single-launch sweep reported a dependency wait that ran
// past its spin limit (resets the sweep state).
static int sweep_error(ilu0_t M, hipStream_t s) {
    rs::SweepCtr c[2];
    HIP_TRY(hipMemcpyAsync(c, M->ctrs.p, sizeof c, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (c[0].error || c[1].error) return sweep_reset(M, s);
    return RS_OK;
}

}  // extern "C"

// Algorithmic bytes of a preconditioner application (equations 3-4), the
// method's minimum whatever the launches: every factor block once with its
// column index (9 tb + 4 bytes, tb = factor element size), a row pointer,
// and the vectors: the lower sweep reads its input and writes y (52 N with
// the row pointer), the upper sweep reads y and writes z (48 N), inv(U_ii)
// counted with U.  Fused work (the p update of an iteration's first lower
// sweep) is not counted.  With one launch per level, the lower launches also
// finish the rows without upper blocks (the upper sweep's first level): their
// inv(U_ii) and z move from the upper sweep's count to the lower one's.
static double fold_bytes(ilu0_t M, double tb) {
    const rs::Schedule &S = M->an->sch;
    if (M->tile_sweeps || S.nu_levels == 0) return 0.0;
    return (9 * tb + 4 + 48.0) * S.uset[1];
}

static double lower_bytes(ilu0_t M, double tb, int nsys) {
    const rs::Schedule &S = M->an->sch;
    return nsys * ((9 * tb + 4) * S.nL + 52.0 * M->n + fold_bytes(M, tb));
}

static double upper_bytes(ilu0_t M, double tb, int nsys) {
    const rs::Schedule &S = M->an->sch;
    return nsys * ((9 * tb + 4) * ((double)S.nU + M->n) + 48.0 * M->n - fold_bytes(M, tb));
}

// Whether an application reads the y of the rows without lower blocks from
// its input instead of storing it (Schedule::y_in): per-level sweeps, and
// the upper launch of those rows reads A' (FP64 factors, or BiCGStab's
// fused iteration), which takes y in FP64.
static bool y_from_input(const rs_ilu0 *M, bool fp64, bool fused) {
    return M->y_input && M->an->sch.y_in && !M->tile_sweeps && (fp64 || fused);
}

// Lower sweep of one preconditioner application M^{-1} in -> out (new
// order).  Timed as one unit (events around its launches).  yin (see
// y_from_input): the first level's rows take y = their input (p, updated
// first, or `in`) and the second level's launch reads it from there.
// Algorithmic bytes of the lower parts: the fused upper launch reads r and
// writes inv(U_kk) r_k and inv(U_kk) v_k on its rows (72 per row); the SpMV
// reads those and writes a_i, b_i (48 per row); the second application's
// lower launch reads s, a, b and inv(U_ii), writes shat (168 per row)
// instead of its L blocks.
static double lp_upper_extra(ilu0_t M, int nsys) { return nsys * 72.0 * M->an->sch.fuse_n0; }
static double lp_spmv_extra(ilu0_t M, int nsys) { return nsys * 48.0 * M->n; }
static double lp_lower_bytes(ilu0_t M, int nsys) { return nsys * 168.0 * (M->n - M->an->sch.fuse_n0); }

template <typename T>
static void lower_levels(ilu0_t M, const T *L, const T *D, const double *in, double *out, bool fuse_p, Krylov &k,
                         SysState *st, int nsys, hipStream_t s, bool prof = true, bool yin = false) {
    const rs::Schedule &S = M->an->sch;
    const size_t vs = k.vstride;
    T *y = (T *)k.y;
    ProfScope ps(PC_LSWEEP, s, lower_bytes(M, sizeof(T), nsys), M->tile_sweeps, prof);
    if (M->tile_sweeps) {
        rs::launch_lsweep_flow<T>(M->an->dev, L, (size_t)S.nL * 9, in, y, out, vs, fuse_p, k.r, k.v, k.p, st, k.lctr,
                                  k.uctr, nsys, S.nl_levels, M->sweep_grid, M->spin_limit, s, ps.start(), ps.stop());
        return;
    }
    // the upper sweep's first level (rows without upper blocks) is finished
    // inside the lower sweep's launches
    const int u0_end = S.nu_levels > 0 ? S.uset[1] : 0;
    if (yin) {
        if (fuse_p) rs::launch_p_update(M->an->dev, k, nsys, s);
        rs::launch_lsweep<T>(M->an->dev, L, (size_t)S.nL * 9, in, y, vs, fuse_p, k.r, k.v, k.p, st, S.lset[1],
                             S.lset[2], nsys, M->sweep_variant, D, (size_t)M->n * 9, out, u0_end,
                             fuse_p ? k.p : in, s);
        return;
    }
    for (int l = 0; l < S.nl_levels; ++l)
        rs::launch_lsweep<T>(M->an->dev, L, (size_t)S.nL * 9, in, y, vs, fuse_p, k.r, k.v, k.p, st, S.lset[l],
                             S.lset[l + 1], nsys, M->sweep_variant, D, (size_t)M->n * 9, out, u0_end, nullptr, s);
}

// Whether BiCGStab's iterations fuse the upper launch of the rows without
// lower blocks with their rows of the SpMV that follows (RS_OPT_FUSE_SPMV).
static bool fused_iteration(const rs_ilu0 *M) {
    return M->fuse_spmv && M->an->sch.fuse_n0 > 0 && !M->tile_sweeps && M->split() == 0;
}

// Algorithmic bytes of the SpMV rows a fused upper launch forms (their
// blocks with column indices, row pointers, x and the product).
static double fused_spmv_bytes(ilu0_t M, int nsys) {
    const rs::Schedule &S = M->an->sch;
    return nsys * (76.0 * (double)S.fuse_nnz + 52.0 * S.fuse_n0);
}

// Whether BiCGStab's iterations form the lower parts of the second
// application inside v = A phat (RS_OPT_LOWER_PARTS): the fused iteration
// on a two-level pattern with FP64 factors, reading y from the input.
static bool lower_parts_iteration(const rs_ilu0 *M) {
    return M->lower_parts && M->precision == RS_PREC_FP64 && fused_iteration(M) && y_from_input(M, true, true) &&
           M->wdev.nw == 0;
}

// Its two workspace vectors, allocated on first use (and kept).
static int ensure_lower_parts(ilu0_t M, hipStream_t s) {
    if (M->lpwork.p) return RS_OK;
    const size_t vec = std::max<size_t>((size_t)M->batch * rs::vec_stride(M->n), 1);
    HIP_TRY(M->lpwork.alloc(2 * vec * sizeof(double)));
    HIP_TRY(hipMemsetAsync(M->lpwork.p, 0, 2 * vec * sizeof(double), s));
    M->k.lp = M->lpwork.as<double>();
    return RS_OK;
}


// Upper sweep levels 1 and up (level 0 is done by the lower sweep), timed
// as one unit.  fmode != FUSE_NONE: the launch of the rows without lower
// blocks also forms their rows of fout = A' out (the product of the
// application's result), with the dot products against fw1.
// yd: the input the rows without lower blocks take as y (when the lower
// sweep ran with yin), else NULL.
// lp: also the lower parts' vectors of the rows without lower blocks
// (lower_parts_iteration, first application).
template <typename T>
static void upper_levels(ilu0_t M, const T *U, const T *D, double *out, bool fuse_p, Krylov &k, SysState *st,
                         int nsys, hipStream_t s, bool prof = true, int fmode = rs::FUSE_NONE,
                         double *fout = nullptr, const double *fw1 = nullptr, const double *yd = nullptr,
                         bool lp = false) {
    const rs::Schedule &S = M->an->sch;
    const size_t vs = k.vstride;
    T *y = (T *)k.y;
    const double fb = (fmode != rs::FUSE_NONE ? fused_spmv_bytes(M, nsys) : 0.0) + (lp ? lp_upper_extra(M, nsys) : 0.0);
    ProfScope ps(PC_USWEEP, s, upper_bytes(M, sizeof(T), nsys) + fb, M->tile_sweeps, prof);
    if (M->tile_sweeps) {
        rs::launch_usweep_flow<T>(M->an->dev, U, (size_t)S.nU * 9, D, (size_t)M->n * 9, y, out, vs, st, k.uctr,
                                  k.lctr, nsys, S.nu_levels, M->sweep_grid, M->spin_limit, s, ps.start(), ps.stop());
        return;
    }
    // the fused rows' upper launch reads their rows of A': always inside
    // BiCGStab's fused iteration, and for every application with FP64
    // factors (whose factorisation stored no U for them)
    const bool via_ap = fmode != rs::FUSE_NONE || (sizeof(T) == sizeof(double) && S.fuse_n0 > 0);
    for (int l = 1; l < S.nu_levels; ++l) {
        int q0 = S.uset[l];
        if (via_ap && l == S.fuse_level) {
            rs::launch_usweep_spmv<T>(M->an->dev, M->pvals.as<double>(), (size_t)M->nnzb * 9, D, (size_t)M->n * 9,
                                      y, yd, out, fout, fw1, st, k, nsys, fmode, M->spmv_variant, fuse_p, s,
                                      nullptr, nullptr, lp);
            q0 += S.fuse_n0;
            if (q0 >= S.uset[l + 1]) continue;
        }
        rs::launch_usweep<T>(M->an->dev, U, (size_t)S.nU * 9, D, (size_t)M->n * 9, y, out, vs, st, q0,
                             S.uset[l + 1], nsys, M->sweep_variant, fuse_p, s);
    }
}

// One preconditioner application M^{-1} in -> out (new order), all levels.
template <typename T>
static void apply_levels(ilu0_t M, const T *L, const T *U, const T *D, const double *in, double *out, bool fuse_p,
                         Krylov &k, SysState *st, int nsys, hipStream_t s, bool prof = true) {
    const double tb = sizeof(T);
    ProfScope ps(PC_APPLY, s, lower_bytes(M, tb, nsys) + upper_bytes(M, tb, nsys), false, prof);
    const bool yin = y_from_input(M, sizeof(T) == sizeof(double), false);
    lower_levels<T>(M, L, D, in, out, fuse_p, k, st, nsys, s, prof, yin);
    upper_levels<T>(M, U, D, out, fuse_p, k, st, nsys, s, prof, rs::FUSE_NONE, nullptr, nullptr,
                    yin ? (fuse_p ? k.p : in) : nullptr);
}

// Parts of a BiCGStab iteration, in order: the two sweeps of the first
// preconditioner application (p updated on the fly), v = A phat, the
// half-step update, the two sweeps of the second application, t = A shat,
// the full-step update.
enum {
    P_L1 = 1, P_U1 = 2, P_SPMV_V = 4, P_SUPD = 8, P_L2 = 16, P_U2 = 32, P_SPMV_T = 64, P_XR = 128, P_ALL = 255
};

// An application is timed as one unit only while neither of its sweeps is
// timed on its own.
static bool apply_unit(int mask) {
    return ((mask >> PC_APPLY) & 1) && !((mask >> PC_LSWEEP) & 1) && !((mask >> PC_USWEEP) & 1);
}

// The iteration parts that hold launches of the kernel classes in `mask`.
static int class_parts(int mask) {
    int parts = 0;
    if ((mask >> PC_LSWEEP) & 1) parts |= P_L1 | P_L2;
    if ((mask >> PC_USWEEP) & 1) parts |= P_U1 | P_U2;
    if (apply_unit(mask)) parts |= P_L1 | P_U1 | P_L2 | P_U2;
    if ((mask >> PC_SPMV_V) & 1) parts |= P_SPMV_V;
    if ((mask >> PC_SPMV_T) & 1) parts |= P_SPMV_T;
    if ((mask >> PC_VEC) & 1) parts |= P_SUPD | P_XR;
    return parts;
}

// Whether a BiCGStab iteration runs each application and its product as one
// launch (k_apply_flow, the same bits): systems of few rows (of all systems),
// whose launches cost more than their bytes, where the launches may be fused
// at all (RS_OPT_FUSE_SPMV) and no sweep or product is timed on its own.
// Solves at reduction 1e-2, one launch against separate ones: 96k cells with
// NNCs, four colours 387 against 436 us, 33 RCM levels 571 against 1 432; four
// colours and 150k cells 473 against 519, 280k cells no faster.  Two-level
// patterns have fewer launches to save: 4 000 cells 177 against 214 us, 20 000
// cells 223 against 233, 50 000 cells 259 against 263 in FP64, 245 against 261
// with FP32 factors.  Not with RS_OPT_USE_GRAPH off, which says that other
// threads solve meanwhile: waiting workgroups hold CUs that the others'
// launches would fill (a burst of 24 requests of 10 000 to 200 000 cells on
// four slots 4.91 against 4.41 ms).  Not on schedules of more than kFlowLevels
// levels either: every level is a hop that all waiting workgroups poll
// through, over all XCDs, and such schedules have the single-launch sweeps
// (RS_OPT_SWEEP_TILES, their default), which run on one.  A 7-point grid of
// 200 000 rows has up to 300 levels under RCM.
constexpr int kFlowLevels = 512;
constexpr long long kFlowRowsMany = 200000, kFlowRowsTwo = 30000, kFlowRowsTwoF32 = 60000;
static bool flow_size(const rs_ilu0 *M, bool wells, bool tiles) {
    const int single = 1 << PC_LSWEEP | 1 << PC_USWEEP | 1 << PC_SPMV_V | 1 << PC_SPMV_T;
    const long long most = !M->an->sch.y_in ? kFlowRowsMany
                           : M->precision == RS_PREC_FP64 ? kFlowRowsTwo : kFlowRowsTwoF32;
    const rs::Schedule &S = M->an->sch;
    return M->use_graph && M->fuse_spmv && !M->no_flow && std::max(S.nl_levels, S.nu_levels) <= kFlowLevels && !tiles && !wells && !(g_prof.mask & single) &&
           (long long)M->n * M->batch <= most;
}
static bool flow_size(const rs_ilu0 *M) { return flow_size(M, M->wdev.nw > 0, M->tile_sweeps); }
static bool flow_iteration(const rs_ilu0 *M) { return flow_size(M) && M->split() == 0; }
// Most workgroups of such a launch: those of large tiles (16 waves of up to
// 128 registers a lane) are resident one a CU, those of small tiles (6 waves)
// one or two; any further ones start as the first leave and find no ticket.
constexpr int kFlowApplyGrid = 512;
// The second y and the second reduction counters of such iterations,
// allocated on first use (and kept).  Where they do not fit the device, the
// handle keeps to the separate launches, which need neither.
static int ensure_flow(ilu0_t M, hipStream_t s, bool &flow) {
    if (!flow || M->ftickets.p) return RS_OK;
    const size_t tb = (size_t)M->batch * M->k.fticket_stride * sizeof(uint32_t);
    hipError_t e = M->ywork2.alloc(std::max<size_t>((size_t)M->batch * rs::vec_stride(M->n), 1) * sizeof(double));
    if (e == hipSuccess) e = M->ftickets.alloc(tb);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        M->no_flow = true;
        flow = false;
        return RS_OK;
    }
    HIP_TRY(e);
    HIP_TRY(hipMemsetAsync(M->ftickets.p, 0, tb, s));
    M->k.y2 = M->ywork2.p;
    M->k.ftickets = M->ftickets.as<uint32_t>();
    return RS_OK;
}

// One such iteration: the first application marks shat and the second y for
// the second application, which marks the first y again; the full-step
// update marks phat.
template <typename T>
static void enqueue_flow_iteration(ilu0_t M, const T *L, const T *U, const T *D, hipStream_t s) {
    Krylov &k = M->k;
    const int B = M->batch, u0_end = M->an->sch.uset[1];
    const double n = M->n, nnzb = M->nnzb, tb = sizeof(T);
    const bool fz = fused_iteration(M);
    const bool lp = sizeof(T) == sizeof(double) && lower_parts_iteration(M);
    const double product = B * (76 * nnzb + 52 * n);
    const double bytes1 = lower_bytes(M, tb, B) + upper_bytes(M, tb, B) + product +
                          (lp ? lp_upper_extra(M, B) + lp_spmv_extra(M, B) : 0.0);
    const double bytes2 = (lp ? lp_lower_bytes(M, B) : lower_bytes(M, tb, B)) + upper_bytes(M, tb, B) + product;
    const double *Ap = M->pvals.as<double>();
    T *ya = (T *)k.y, *yb = (T *)k.y2;
    {
        ProfScope ps(PC_APPLY, s, bytes1, true);
        rs::launch_apply_flow<T>(M->an->dev, L, U, D, Ap, nullptr, ya, yb, k.phat, k.shat, k.v, k.rhat, k, k.st,
                                 k.lctr, k.uctr, u0_end, B, rs::APPLY_V, fz, lp, M->spmv_variant, M->an->sch.nl_levels, kFlowApplyGrid,
                                 M->spin_limit, s, ps.start(), ps.stop());
    }
    {
        ProfScope ps(PC_VEC, s, B * 72 * n, true);
        rs::launch_s_update(M->an->dev, k, B, M->spmv_variant, 0, fz, s, ps.start(), ps.stop());
    }
    {
        ProfScope ps(PC_APPLY, s, bytes2, true);
        rs::launch_apply_flow<T>(M->an->dev, L, U, D, Ap, k.s, yb, ya, k.shat, nullptr, k.t, k.s, k, k.st, k.uctr,
                                 k.lctr, u0_end, B, rs::APPLY_T, fz, lp, M->spmv_variant, M->an->sch.nl_levels, kFlowApplyGrid,
                                 M->spin_limit, s, ps.start(), ps.stop());
    }
    {
        ProfScope ps(PC_VEC, s, B * 192 * n, true);
        rs::launch_xr_update(M->an->dev, k, B, M->spmv_variant, 0, fz, s, ps.start(), ps.stop(), false, true);
    }
}

template <typename T>
static void enqueue_iteration(ilu0_t M, const T *L, const T *U, const T *D, hipStream_t s, int parts) {
    if (parts == P_ALL && flow_iteration(M)) {
        enqueue_flow_iteration<T>(M, L, U, D, s);
        return;
    }
    Krylov &k = M->k;
    const int B = M->batch;
    const size_t per = (size_t)M->nnzb * 9;
    const double n = M->n, nnzb = M->nnzb, tb = sizeof(T);
    // algorithmic bytes of y = A x: values and column indices, row
    // pointers, x read once, y written (the fused dot product's second
    // vector is not counted)
    // with the fused upper launch, the rows without lower blocks of v and t
    // (and their bytes) move from the SpMV into the application
    const bool fz = fused_iteration(M);
    const bool yin = y_from_input(M, sizeof(T) == sizeof(double), fz);
    const bool lp = sizeof(T) == sizeof(double) && lower_parts_iteration(M);
    const int r0 = fz ? M->an->sch.fuse_n0 : 0;
    // wells with the fused iteration: the fused rows' well terms come after
    // each product, with one more group sum for the vector kernels
    const bool wfix = fz && M->wdev.nw > 0 && M->wdev.nfix > 0;
    const int fix_at = wfix ? rs::wells_fix_at(M->an->dev, M->spmv_variant) : 0;
    const double fb = fz ? fused_spmv_bytes(M, B) : 0.0;
    const double spmv_bytes = B * (76 * nnzb + 52 * n) - fb;
    const double apply_bytes = lower_bytes(M, tb, B) + upper_bytes(M, tb, B) + fb;
    {
        // an application is timed whole or not at all
        ProfScope pa(PC_APPLY, s, apply_bytes + (lp ? lp_upper_extra(M, B) : 0.0), false,
                     (parts & P_L1) && (parts & P_U1));
        if (parts & P_L1) lower_levels<T>(M, L, D, nullptr, k.phat, true, k, k.st, B, s, true, yin);
        if (parts & P_U1)
            upper_levels<T>(M, U, D, k.phat, true, k, k.st, B, s, true, fz ? rs::FUSE_V : rs::FUSE_NONE, k.v,
                            k.rhat, yin ? k.p : nullptr, lp);
    }
    if (parts & P_SPMV_V) {
        ProfScope ps(PC_SPMV_V, s, spmv_bytes + (lp ? lp_spmv_extra(M, B) : 0.0), true);
        if (lp)
            rs::launch_spmv_lp(M->an->dev, M->pvals.as<double>(), per, k, B, M->spmv_variant, s, ps.start(),
                               ps.stop());
        else
            rs::launch_spmv_v(M->an->dev, M->pvals.as<double>(), per, k, B, M->spmv_variant, M->split(), M->wdev,
                              r0, s, ps.start(), ps.stop());
        // the well terms of the rows the fused upper launch formed
        if (wfix) rs::launch_wells_fix(M->wdev, k.v, k.rhat, k.vstride, k.fpart, k.fpart_stride, fix_at, k.st, B, s);
    }
    if (parts & P_SUPD) {
        ProfScope ps(PC_VEC, s, B * 72 * n, true);
        rs::launch_s_update(M->an->dev, k, B, M->spmv_variant, M->split(), fz, s, ps.start(), ps.stop(), wfix);
    }
    {
        ProfScope pa(PC_APPLY, s, lp ? lp_lower_bytes(M, B) + upper_bytes(M, tb, B) + fb : apply_bytes, false,
                     (parts & P_L2) && (parts & P_U2));
        if ((parts & P_L2) && lp) {
            // the second level's rows from the SpMV's lower parts; the first
            // level's y is s itself
            ProfScope pl(PC_LSWEEP, s, lp_lower_bytes(M, B), false);
            rs::launch_lower_parts(M->an->dev, (const double *)D, (size_t)M->n * 9, k, B, s);
        } else if (parts & P_L2) {
            lower_levels<T>(M, L, D, k.s, k.shat, false, k, k.st, B, s, true, yin);
        }
        if (parts & P_U2)
            upper_levels<T>(M, U, D, k.shat, false, k, k.st, B, s, true, fz ? rs::FUSE_T : rs::FUSE_NONE, k.t,
                            k.s, yin ? k.s : nullptr);
    }
    if (parts & P_SPMV_T) {
        ProfScope ps(PC_SPMV_T, s, spmv_bytes, true);
        rs::launch_spmv_t(M->an->dev, M->pvals.as<double>(), per, k, B, M->spmv_variant, M->split(), M->wdev, r0,
                          s, ps.start(), ps.stop());
        if (wfix) rs::launch_wells_fix(M->wdev, k.t, k.s, k.vstride, k.fpart, k.fpart_stride, fix_at, k.st, B, s);
    }
    if (parts & P_XR) {
        ProfScope ps(PC_VEC, s, B * 192 * n, true);
        rs::launch_xr_update(M->an->dev, k, B, M->spmv_variant, M->split(), fz, s, ps.start(), ps.stop(), wfix);
    }
}

static void enqueue_iteration_any(ilu0_t M, hipStream_t s, int parts) {
    if (M->precision == RS_PREC_FP32_FACTORS)
        enqueue_iteration<float>(M, M->Lf.as<float>(), M->Uf.as<float>(), M->Dinvf.as<float>(), s, parts);
    else
        enqueue_iteration<double>(M, M->L.as<double>(), M->U.as<double>(), M->Dinv.as<double>(), s, parts);
}

// Replay the graph segment holding `parts` (captured on a private stream
// the first time this configuration is seen).  Nothing is timed inside a
// graph: profiling is off while segments are captured.
// A graph segment of `reps` consecutive whole iterations is keyed as parts
// P_ALL + (reps - 1) * kRepShift.
constexpr int kRepShift = 1 << 16;

static int replay_segment(ilu0_t M, int parts, hipStream_t s, int reps = 1) {
    rs_ilu0::GraphKey key;
    key.precision = M->precision;
    key.tile_sweeps = M->tile_sweeps;
    key.spmv_variant = M->spmv_variant;
    key.sweep_variant = M->sweep_variant;
    key.split = M->split();
    key.sweep_grid = M->sweep_grid;
    key.spin = M->spin_limit;
    key.fuse = fused_iteration(M) ? 1 : 0;
    key.yin = M->y_input ? 1 : 0;
    key.lp = M->lower_parts ? 1 : 0;
    key.flow = parts == P_ALL && flow_iteration(M) ? 1 : 0;
    key.wells = M->wdev.nw > 0 ? (long long)M->wells_version + 1 : 0;
    rs_ilu0::Segment &seg = M->segments[parts + (reps - 1) * kRepShift];
    if (!seg.exec || !(seg.key == key)) {
        if (seg.exec) (void)hipGraphExecDestroy(seg.exec);
        if (seg.graph) (void)hipGraphDestroy(seg.graph);
        seg.exec = nullptr;
        seg.graph = nullptr;
        if (!M->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&M->cap_stream, hipStreamNonBlocking));
        const int mask = g_prof.mask;
        g_prof.mask = 0;
        hipError_t e = hipStreamBeginCapture(M->cap_stream, hipStreamCaptureModeRelaxed);
        if (e == hipSuccess) {
            for (int i = 0; i < reps; ++i) enqueue_iteration_any(M, M->cap_stream, parts);
            e = hipStreamEndCapture(M->cap_stream, &seg.graph);
        }
        g_prof.mask = mask;
        HIP_TRY(e);
        HIP_TRY(hipGraphInstantiate(&seg.exec, seg.graph, nullptr, nullptr, 0));
        seg.key = key;
    }
    HIP_TRY(hipGraphLaunch(seg.exec, s));
    return RS_OK;
}

// Queue one BiCGStab iteration on `s`.  With graphs on, the iteration is
// one replay.  While kernel classes are timed, each of their parts is timed
// on its own: a per-level sweep replays as a graph segment of its own
// between two events (the unit is the whole sweep), a single launch runs
// directly and records dispatch events; the runs of untimed parts between
// them replay as graph segments.
static int run_iteration(ilu0_t M, hipStream_t s) {
    if (!M->use_graph) {
        enqueue_iteration_any(M, s, P_ALL);
        HIP_TRY(hipGetLastError());
        return RS_OK;
    }
    const int timed = class_parts(g_prof.mask);
    if (!timed) return replay_segment(M, P_ALL, s);
    if (flow_iteration(M)) {
        // every launch is a unit of its own: its events come with the dispatch
        enqueue_iteration_any(M, s, P_ALL);
        HIP_TRY(hipGetLastError());
        return RS_OK;
    }
    const double tb = M->precision == RS_PREC_FP32_FACTORS ? 4 : 8;
    // the SpMV rows a fused upper launch forms count with the application
    const double fb = fused_iteration(M) ? fused_spmv_bytes(M, M->batch) : 0.0;
    const bool lp = lower_parts_iteration(M);
    // per part: the first application's upper launch also forms the lower
    // parts' vectors; the second application's lower launch reads them
    auto lo_bytes = [&](int part) {
        return lp && part == P_L2 ? lp_lower_bytes(M, M->batch) : lower_bytes(M, tb, M->batch);
    };
    auto up_bytes = [&](int part) {
        return upper_bytes(M, tb, M->batch) + fb + (lp && part == P_U1 ? lp_upper_extra(M, M->batch) : 0.0);
    };
    const bool whole = apply_unit(g_prof.mask);
    int run = 0;
    for (int part = 1; part <= P_XR; part <<= 1) {
        if (!(timed & part)) {
            run |= part;
            continue;
        }
        if (run) {
            const int st = replay_segment(M, run, s);
            if (st != RS_OK) return st;
            run = 0;
        }
        if (whole && (part == P_L1 || part == P_L2)) {
            // a whole application (both sweeps) as one graph segment between two events
            ProfScope ps(PC_APPLY, s, lo_bytes(part) + up_bytes(part << 1));
            const int st = replay_segment(M, part | (part << 1), s);
            if (st != RS_OK) return st;
            part <<= 1;   // its upper sweep is done
            continue;
        }
        const bool sweep = part == P_L1 || part == P_U1 || part == P_L2 || part == P_U2;
        if (sweep && !M->tile_sweeps) {
            const bool lower = part == P_L1 || part == P_L2;
            ProfScope ps(lower ? PC_LSWEEP : PC_USWEEP, s, lower ? lo_bytes(part) : up_bytes(part));
            const int st = replay_segment(M, part, s);
            if (st != RS_OK) return st;
        } else {
            enqueue_iteration_any(M, s, part);
            HIP_TRY(hipGetLastError());
        }
    }
    return run ? replay_segment(M, run, s) : RS_OK;
}

// Queue `count` BiCGStab iterations on `s`.  Without kernel-class timing,
// runs of 8, 4, 2 and 1 whole iterations replay as one graph each: the
// launches inside a graph follow one another with no gap, while every graph
// launch costs a few microseconds of idle device time at its boundary.
static int run_iterations(ilu0_t M, int count, hipStream_t s) {
    if (M->use_graph && !class_parts(g_prof.mask)) {
        for (int reps = 8; reps >= 1; reps >>= 1)
            while (count >= reps) {
                const int st = replay_segment(M, P_ALL, s, reps);
                if (st != RS_OK) return st;
                count -= reps;
            }
        return RS_OK;
    }
    for (int i = 0; i < count; ++i) {
        const int st = run_iteration(M, s);
        if (st != RS_OK) return st;
    }
    return RS_OK;
}

extern "C" {

int ilu0_apply(ilu0_t M, const double *v, double *z, int32_t first_sys, int32_t n_sys, int32_t mem, void *stream) {
    if (!M || !v || !z || first_sys < 0 || n_sys < 0 || first_sys + n_sys > M->batch)
        return fail(RS_INVALID_ARG, "ilu0_apply: bad arguments");
    if (!M->factored) return fail(RS_NOT_FACTORED, "ilu0_apply: not factored");
    if (n_sys == 0 || M->n == 0) return RS_OK;
    hipStream_t s = (hipStream_t)stream;
    int st = refuse_capture(s, "ilu0_apply");
    if (st != RS_OK) return st;
    if ((st = after_apply(M, s)) != RS_OK) return st;
    if ((st = ensure_workspace(M, s)) != RS_OK) return st;
    const bool fills_u = reads_u(M, false) && M->u_missing;
    if (fills_u && (st = ensure_u(M, s)) != RS_OK) return st;
    const size_t m = 3 * (size_t)M->n * n_sys;
    const double *vd = nullptr;
    st = stage_in(v, mem, M->bstage, m, s, &vd);
    if (st != RS_OK) return st;
    double *zd = z;
    if (mem != RS_MEM_DEVICE) {
        HIP_TRY(M->xstage.alloc(m * sizeof(double)));
        zd = M->xstage.as<double>();
    }
    Krylov &k = M->k;
    const rs::Schedule &S = M->an->sch;
    rs::launch_permute_vec(M->an->dev.perm, vd, k.s, M->n, k.vstride, n_sys, false, s);
    if (M->precision == RS_PREC_FP32_FACTORS)
        apply_levels<float>(M, M->Lf.as<float>() + (size_t)first_sys * S.nL * 9,
                            M->Uf.as<float>() + (size_t)first_sys * S.nU * 9,
                            M->Dinvf.as<float>() + (size_t)first_sys * M->n * 9, k.s, k.shat, false, k, nullptr,
                            n_sys, s);
    else
        apply_levels<double>(M, M->L.as<double>() + (size_t)first_sys * S.nL * 9,
                             M->U.as<double>() + (size_t)first_sys * S.nU * 9,
                             M->Dinv.as<double>() + (size_t)first_sys * M->n * 9, k.s, k.shat, false, k, nullptr,
                             n_sys, s);
    rs::launch_permute_vec(M->an->dev.perm, k.shat, zd, M->n, k.vstride, n_sys, true, s);
    HIP_TRY(hipGetLastError());
    if (mem != RS_MEM_DEVICE) HIP_TRY(hipMemcpyAsync(z, zd, m * sizeof(double), hipMemcpyDeviceToHost, s));
    // Only single-launch sweeps leave a word to read, and host vectors need
    // the copy's end; a device caller's stream goes on without the host
    // (200 000 cells, an application and a product: 99 -> 74 us).  An event
    // keeps the handle's next call behind this one.  The one application of a
    // factorisation that fills in U waits for it, so that other streams (and
    // captures, which cannot wait for the event) find it in place.
    if (M->tile_sweeps || mem != RS_MEM_DEVICE) return sweep_error(M, s);
    if (fills_u) HIP_TRY(hipStreamSynchronize(s));
    if (!M->ev_apply) HIP_TRY(hipEventCreateWithFlags(&M->ev_apply, hipEventDisableTiming));
    HIP_TRY(hipEventRecord(M->ev_apply, s));
    M->apply_stream = s;
    M->apply_queued = true;
    return RS_OK;
}

}  // extern "C"

// ------------------------------------------------------ allocation-free apply

// Workspace of ilu0_apply_noalloc: one file-scope array per GPU, held until
// the process ends.  On the host, `scratch` names a stand-in, not device
// memory: host code uses only the address hipGetSymbolAddress returns for
// the current device (noalloc_scratch), never the name itself.
static __device__ __align__(256) unsigned char scratch[RS_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's `scratch`, looked up once per
// device with that device current.
int noalloc_scratch(unsigned char **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(RS_HIP_ERROR, "ilu0_apply_noalloc: device ordinal out of range");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(RS_HIP_ERROR, "ilu0_apply_noalloc: no device address for the workspace");
        g_scratch_ptr[dev] = p;
    }
    *out = (unsigned char *)g_scratch_ptr[dev];
    return RS_OK;
}

// Carving of the workspace for n_sys systems of M: the new-order input, the
// lower sweep's y, the new-order output (each n_sys * vstride doubles), and
// the single-launch sweeps' two counters; each part 256-byte aligned.
struct NoAllocLayout {
    size_t vin, y, vout, ctrs, end;
};

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

NoAllocLayout noalloc_layout(const rs_ilu0 *M, int n_sys) {
    NoAllocLayout l{};
    const size_t vec = align256((size_t)n_sys * rs::vec_stride(M->n) * sizeof(double));
    l.vin = 0;
    l.y = vec;
    l.vout = 2 * vec;
    l.ctrs = 3 * vec;
    l.end = l.ctrs + align256(2 * sizeof(rs::SweepCtr));
    return l;
}

}  // namespace

extern "C" {

int ilu0_apply_noalloc(ilu0_t M, const double *v, double *z, int32_t first_sys, int32_t n_sys, void *stream) {
    if (!M || !v || !z || first_sys < 0 || n_sys < 0 || first_sys + n_sys > M->batch)
        return fail(RS_INVALID_ARG, "ilu0_apply_noalloc: bad arguments");
    if (!M->factored) return fail(RS_NOT_FACTORED, "ilu0_apply_noalloc: not factored");
    if (n_sys == 0 || M->n == 0) return RS_OK;
    const NoAllocLayout lay = noalloc_layout(M, n_sys);
    if (lay.end > (size_t)RS_NOALLOC_SCRATCH_BYTES)
        return fail(RS_OUT_OF_MEMORY, "ilu0_apply_noalloc: " + std::to_string(n_sys) + " system(s) of " +
                                          std::to_string(M->n) + " block rows need " + std::to_string(lay.end) +
                                          " bytes of workspace, above its fixed size of " +
                                          std::to_string((size_t)RS_NOALLOC_SCRATCH_BYTES));
    unsigned char *base = nullptr;
    int st = noalloc_scratch(&base);
    if (st != RS_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    // shares with the handle's queued applications only the factors, which
    // those leave whole (see ilu0_apply)
    if (reads_u(M, false) && (st = ensure_u(M, s)) != RS_OK) return st;
    Krylov k{};
    k.vstride = rs::vec_stride(M->n);
    double *vin = (double *)(base + lay.vin), *vout = (double *)(base + lay.vout);
    k.y = base + lay.y;
    k.lctr = (rs::SweepCtr *)(base + lay.ctrs);
    k.uctr = k.lctr + 1;
    // the workspace keeps the last call's contents (any handle's): the
    // single-launch sweeps' counters and marks are set anew
    if (M->tile_sweeps) {
        rs::launch_fill_u32((uint32_t *)(base + lay.ctrs), (lay.end - lay.ctrs) / sizeof(uint32_t), 0u, s);
        rs::launch_flow_mark(k.y, lay.vout - lay.y, s);
    }
    const rs::Schedule &S = M->an->sch;
    rs::launch_permute_vec(M->an->dev.perm, v, vin, M->n, k.vstride, n_sys, false, s);
    if (M->precision == RS_PREC_FP32_FACTORS)
        apply_levels<float>(M, M->Lf.as<float>() + (size_t)first_sys * S.nL * 9,
                            M->Uf.as<float>() + (size_t)first_sys * S.nU * 9,
                            M->Dinvf.as<float>() + (size_t)first_sys * M->n * 9, vin, vout, false, k, nullptr,
                            n_sys, s, false);
    else
        apply_levels<double>(M, M->L.as<double>() + (size_t)first_sys * S.nL * 9,
                             M->U.as<double>() + (size_t)first_sys * S.nU * 9,
                             M->Dinv.as<double>() + (size_t)first_sys * M->n * 9, vin, vout, false, k, nullptr,
                             n_sys, s, false);
    rs::launch_permute_vec(M->an->dev.perm, vout, z, M->n, k.vstride, n_sys, true, s);
    HIP_TRY(hipGetLastError());
    if (!M->tile_sweeps) return RS_OK;
    // a single-launch sweep whose dependency wait gave up leaves its error word set
    rs::SweepCtr c[2];
    HIP_TRY(hipMemcpyAsync(c, k.lctr, sizeof c, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (c[0].error || c[1].error)
        return fail(RS_HIP_ERROR, "ilu0_apply_noalloc: sweep dependency wait exceeded its limit");
    return RS_OK;
}

static int status_rank(int s) {
    if (s == RS_HIP_ERROR) return 5;   // a queued factorisation's wait gave up
    if (s < 0) return 4;
    if (s == RS_BREAKDOWN) return 3;
    if (s == RS_NOT_CONVERGED) return 2;
    return 1;
}

int bicgstab_solve(ilu0_t M, bcsr_t A, const double *b, double *x, double reduction, int32_t max_iter, int32_t mem,
                   void *stream, solve_info *info) {
    int st = check_pair(M, A);
    if (st != RS_OK) return st;
    if (!b || !x || !(reduction >= 0.0) || max_iter < 0 || (mem != RS_MEM_HOST && mem != RS_MEM_DEVICE))
        return fail(RS_INVALID_ARG, "bicgstab_solve: bad arguments");
    if (!M->factored) return fail(RS_NOT_FACTORED, "bicgstab_solve: call ilu0_factor first");
    const int B = M->batch;
    if (M->n == 0) {
        if (info)
            for (int i = 0; i < B; ++i) info[i] = solve_info{RS_OK, 0, 0.0, 0.0, 0.0, factor_time(M), 0.0};
        return RS_OK;
    }
    hipStream_t s = (hipStream_t)stream;
    if ((st = refuse_capture(s, "bicgstab_solve")) != RS_OK) return st;
    if ((st = after_apply(M, s)) != RS_OK) return st;
    st = ensure_workspace(M, s);
    if (st != RS_OK) return st;
    st = ensure_wells(M, A, s);
    if (st != RS_OK) return st;
    bool flow = flow_iteration(M);
    if ((st = ensure_flow(M, s, flow)) != RS_OK) return st;
    if (!flow && reads_u(M, fused_iteration(M)) && (st = ensure_u(M, s)) != RS_OK) return st;
    if (lower_parts_iteration(M) && (st = ensure_lower_parts(M, s)) != RS_OK) return st;
    const size_t m = 3 * (size_t)M->n * B;
    const double *bd = nullptr;
    st = stage_in(b, mem, M->bstage, m, s, &bd);
    if (st != RS_OK) return st;
    double *xd = x;
    if (mem != RS_MEM_DEVICE) {
        HIP_TRY(M->xstage.alloc(m * sizeof(double)));
        xd = M->xstage.as<double>();
    }
    Krylov &k = M->k;
    st = solve_events(M, s);
    if (st != RS_OK) return st;
    {
        ProfScope ps(PC_VEC, s, (double)B * 152 * M->n);
        rs::launch_setup(M->an->dev, bd, M->bad.as<int32_t>(), reduction, max_iter, k, B, flow, s);
    }
    // x back to the caller's order, the true residual, and the results to the host
    auto finish = [&]() -> int {
        rs::launch_finish(M->an->dev, A->rowptr.as<int32_t>(), A->colidx.as<int32_t>(), A->vals.as<double>(),
                          (size_t)A->nnzb * 9, bd, xd, k, B, M->spmv_variant, M->split(), A->wells(), s);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipEventRecord(M->ev_s1, s));
        HIP_TRY(hipMemcpyAsync(M->h_state, k.st, B * sizeof(SysState), hipMemcpyDeviceToHost, s));
        // only single-launch sweeps and applications touch the counters
        if (M->tile_sweeps || flow) HIP_TRY(hipMemcpyAsync(M->h_ctr, k.lctr, 2 * sizeof(rs::SweepCtr), hipMemcpyDeviceToHost, s));
        if (mem != RS_MEM_DEVICE) HIP_TRY(hipMemcpyAsync(x, xd, m * sizeof(double), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        M->apply_queued = false;   // `s` came after it
        return RS_OK;
    };
    auto all_done = [&]() {
        bool all = true;
        for (int i = 0; i < B; ++i) all &= (M->h_state[i].phase == rs::PH_DONE);
        return all;
    };
    // The first poll comes after as many iterations as the previous solve
    // needed and carries the finishing work with it, so a solve that ends
    // there costs one host synchronisation; otherwise the finishing work is
    // simply repeated after the last iteration.
    int done_iters = 0;
    bool first = true, finished = false;
    while (done_iters < max_iter) {
        const bool predicted = first && M->predict;
        int c = predicted ? std::max(M->chunk, M->last_iters) : M->chunk;
        c = std::min(c, max_iter - done_iters);
        first = false;
        st = run_iterations(M, c, s);
        if (st != RS_OK) return st;
        done_iters += c;
        if (predicted) {
            st = finish();
            if (st != RS_OK) return st;
            if (all_done()) {
                finished = true;
                break;
            }
            continue;
        }
        HIP_TRY(hipMemcpyAsync(M->h_state, k.st, B * sizeof(SysState), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        if (all_done()) break;
    }
    if (!finished) {
        st = finish();
        if (st != RS_OK) return st;
    }
    if ((st = solve_waits(M, M->tile_sweeps || flow, s)) != RS_OK) return st;
    const double solve_ms = elapsed_ms(M->ev_s0, M->ev_s1);
    int worst = RS_OK, needed = 1;
    for (int i = 0; i < B; ++i) {
        const SysState &S = M->h_state[i];
        if (info) info[i] = solve_info{S.status, S.half_steps, S.r0norm, S.last_norm, S.true_res, factor_time(M), solve_ms};
        if (status_rank(S.status) > status_rank(worst)) worst = S.status;
        needed = std::max(needed, (S.half_steps + 1) / 2);
    }
    // the prediction learns from converged solves only, and stays small
    if (worst == RS_OK) M->last_iters = std::min(needed, kPredictMax);
    if (worst == RS_HIP_ERROR) factor_message(worst);
    return worst;
}

}  // extern "C"

// GMRES steps use the fused upper launch where BiCGStab's iteration would
// (RS_OPT_FUSE_SPMV).
static bool gm_fused(const rs_ilu0 *M) {
    return M->fuse_spmv && M->an->sch.fuse_n0 > 0 && !M->tile_sweeps;
}

// The vectors of GMRES's single-launch applications: two pairs (y, z) used in
// turn, each launch marking the other pair for the next one.  (A system that
// stops skips the launches that follow, so after a cycle's end both start
// anew from a marked pair.)
struct GmFlow {
    bool on = false;
    int pair = 0;   // the pair that is marked
    int ctr = 0;    // the counter that is clear (each launch clears the other)
};

// One such launch: z = M^-1 in and, with mode APPLY_RUN, k.t = A' z.
// Returns z.
template <typename T>
static double *gm_apply_flow(ilu0_t M, const T *L, const T *U, const T *D, const double *in, SysState *st, int mode,
                             GmFlow &f, hipStream_t s, const ProfScope &ps) {
    Krylov &k = M->k;
    T *y[2] = {(T *)k.y, (T *)k.y2};
    double *z[2] = {k.phat, k.shat};
    rs::SweepCtr *c[2] = {k.lctr, k.uctr};
    const int p = f.pair, q = f.ctr;
    f.pair = 1 - p;
    f.ctr = 1 - q;
    rs::launch_apply_flow<T>(M->an->dev, L, U, D, M->pvals.as<double>(), in, y[p], y[1 - p], z[p], z[1 - p], k.t,
                             nullptr, k, st, c[q], c[1 - q], M->an->sch.uset[1], M->batch, mode, gm_fused(M), false,
                             M->spmv_variant, M->an->sch.nl_levels, kFlowApplyGrid, M->spin_limit, s, ps.start(),
                             ps.stop());
    return z[p];
}

// Queue one Arnoldi step (column j) of every iterating system on `s`.
// Timed launches record their own dispatch events.
template <typename T>
static void gm_step(ilu0_t M, const T *L, const T *U, const T *D, const rs::GmWork &g, int j, GmFlow &flow,
                    hipStream_t s) {
    Krylov &k = M->k;
    const int B = M->batch;
    const double n = M->n, nnzb = M->nnzb, vb = (double)B * 24 * n;
    // z = M^-1 v_j, w = A z; with the fused upper launch (as in BiCGStab's
    // iteration) the rows without lower blocks form their rows of w there
    // (the launch's dot products go unused) and the SpMV covers the others
    const double *vj = g.V + (size_t)j * g.colstride;
    const bool fz = gm_fused(M);
    const double fb = fz ? fused_spmv_bytes(M, B) : 0.0;
    if (flow.on) {
        ProfScope ps(PC_APPLY, s,
                     lower_bytes(M, sizeof(T), B) + upper_bytes(M, sizeof(T), B) + B * (76 * nnzb + 52 * n), true);
        gm_apply_flow<T>(M, L, U, D, vj, k.st, rs::APPLY_RUN, flow, s, ps);
    } else if (fz) {
        const bool yin = y_from_input(M, sizeof(T) == sizeof(double), true);
        ProfScope ps(PC_APPLY, s, lower_bytes(M, sizeof(T), B) + upper_bytes(M, sizeof(T), B) + fb, false, true);
        lower_levels<T>(M, L, D, vj, k.phat, false, k, k.st, B, s, true, yin);
        upper_levels<T>(M, U, D, k.phat, false, k, k.st, B, s, true, rs::FUSE_V, k.t, vj, yin ? vj : nullptr);
    } else {
        apply_levels<T>(M, L, U, D, vj, k.phat, false, k, k.st, B, s);
    }
    if (!flow.on) {
        ProfScope ps(PC_SPMV_T, s, B * (76 * nnzb + 4 * n + 48 * n) - fb, true);
        rs::launch_spmv_running(M->an->dev, M->pvals.as<double>(), (size_t)M->nnzb * 9, k.phat, k.t, k.vstride, k.st,
                                B, M->spmv_variant, M->wdev, s, ps.start(), ps.stop(),
                                fz ? M->an->sch.fuse_n0 : 0);
        // the well terms of the rows the fused launch formed (the dot
        // products of w come later, from the finished w: the fix-up's sums
        // go unused)
        if (fz && M->wdev.nw > 0 && M->wdev.nfix > 0)
            rs::launch_wells_fix(M->wdev, k.t, vj, k.vstride, k.fpart, k.fpart_stride,
                                 rs::wells_fix_at(M->an->dev, M->spmv_variant), k.st, B, s);
    }
    const int jv = j + 1;
    {
        ProfScope ps(PC_GM, s, vb * (jv + 1), true);
        rs::launch_gm_dots(g, jv, k.t, M->n, B, s, ps.start(), ps.stop());
    }
    {
        ProfScope ps(PC_GM, s, vb * (jv + 2), true);
        rs::launch_gm_orth(g, jv, k.t, false, M->n, B, s, ps.start(), ps.stop());
    }
    {
        ProfScope ps(PC_GM, s, vb * (jv + 2), true);
        rs::launch_gm_orth(g, jv, k.t, true, M->n, B, s, ps.start(), ps.stop());
    }
}

// End of a cycle: x += M^-1 (V y) for every system not done, then the
// restart of those still iterating from r = P b - A x.
template <typename T>
static void gm_cycle_end(ilu0_t M, const T *L, const T *U, const T *D, const rs::GmWork &g, int cols, GmFlow &flow,
                         hipStream_t s) {
    Krylov &k = M->k;
    const int B = M->batch;
    const double n = M->n, nnzb = M->nnzb, vb = (double)B * 24 * n;
    {
        // (cols = steps queued in the cycle, an upper bound of every system's basis)
        ProfScope ps(PC_VEC, s, vb * (cols + 1), true);
        rs::launch_gm_combine(g, k.s, M->n, B, s, ps.start(), ps.stop());
    }
    const double *z = k.phat;
    if (flow.on) {
        // both counters clear: the launch takes the second and so leaves the
        // first clear, as the next cycle and the next solve find it
        flow.pair = 0;
        flow.ctr = 1;
        rs::launch_flow_pair(k, M->n, B, s);
        ProfScope ps(PC_APPLY, s, lower_bytes(M, sizeof(T), B) + upper_bytes(M, sizeof(T), B), true);
        z = gm_apply_flow<T>(M, L, U, D, k.s, nullptr, rs::APPLY_ONLY, flow, s, ps);
    } else {
        apply_levels<T>(M, L, U, D, k.s, k.phat, false, k, nullptr, B, s);
    }
    {
        ProfScope ps(PC_VEC, s, vb * 3, true);
        rs::launch_gm_xupdate(g, k.x, z, M->n, B, s, ps.start(), ps.stop());
    }
    rs::launch_gm_phase(g, B, s);
    {
        ProfScope ps(PC_SPMV_T, s, B * (76 * nnzb + 4 * n + 48 * n), true);
        rs::launch_spmv_running(M->an->dev, M->pvals.as<double>(), (size_t)M->nnzb * 9, k.x, k.t, k.vstride, k.st, B,
                                M->spmv_variant, M->wdev, s, ps.start(), ps.stop());
    }
    {
        ProfScope ps(PC_VEC, s, vb * 3, true);
        rs::launch_gm_restart(g, k.rhat, k.t, k.r, M->n, B, s, ps.start(), ps.stop());
    }
    {
        ProfScope ps(PC_VEC, s, vb * 2, true);
        rs::launch_gm_normalise(g, k.r, 0, 0, M->n, B, s, ps.start(), ps.stop());
    }
}

static void gm_step_any(ilu0_t M, const rs::GmWork &g, int j, GmFlow &flow, hipStream_t s) {
    if (M->precision == RS_PREC_FP32_FACTORS)
        gm_step<float>(M, M->Lf.as<float>(), M->Uf.as<float>(), M->Dinvf.as<float>(), g, j, flow, s);
    else
        gm_step<double>(M, M->L.as<double>(), M->U.as<double>(), M->Dinv.as<double>(), g, j, flow, s);
}

static void gm_cycle_end_any(ilu0_t M, const rs::GmWork &g, int cols, GmFlow &flow, hipStream_t s) {
    if (M->precision == RS_PREC_FP32_FACTORS)
        gm_cycle_end<float>(M, M->Lf.as<float>(), M->Uf.as<float>(), M->Dinvf.as<float>(), g, cols, flow, s);
    else
        gm_cycle_end<double>(M, M->L.as<double>(), M->U.as<double>(), M->Dinv.as<double>(), g, cols, flow, s);
}

extern "C" {

int gmres_solve(ilu0_t M, bcsr_t A, const double *b, double *x, int32_t restart, double reduction, int32_t max_iter,
                int32_t mem, void *stream, solve_info *info) {
    int st = check_pair(M, A);
    if (st != RS_OK) return st;
    if (!b || !x || !(reduction >= 0.0) || max_iter < 0 || restart < 1 || restart > rs::kGmMax ||
        (mem != RS_MEM_HOST && mem != RS_MEM_DEVICE))
        return fail(RS_INVALID_ARG, "gmres_solve: bad arguments");
    if (!M->factored) return fail(RS_NOT_FACTORED, "gmres_solve: call ilu0_factor first");
    const int B = M->batch;
    if (M->n == 0) {
        if (info)
            for (int i = 0; i < B; ++i) info[i] = solve_info{RS_OK, 0, 0.0, 0.0, 0.0, factor_time(M), 0.0};
        return RS_OK;
    }
    hipStream_t s = (hipStream_t)stream;
    if ((st = refuse_capture(s, "gmres_solve")) != RS_OK) return st;
    if ((st = after_apply(M, s)) != RS_OK) return st;
    st = ensure_workspace(M, s);
    if (st != RS_OK) return st;
    st = ensure_wells(M, A, s);
    if (st != RS_OK) return st;
    GmFlow flow;
    flow.on = flow_size(M);
    if ((st = ensure_flow(M, s, flow.on)) != RS_OK) return st;
    if (!flow.on && reads_u(M, false) && (st = ensure_u(M, s)) != RS_OK) return st;
    Krylov &k = M->k;
    // basis: restart columns (the column a cycle's last step would add is
    // never used); zeroed once, so the padding of every column stays zero
    const size_t colstride = (size_t)B * k.vstride;
    const size_t basis_bytes = (size_t)restart * colstride * sizeof(double);
    if (!M->gm_basis.p || M->gm_basis.bytes < basis_bytes) {
        HIP_TRY(M->gm_basis.alloc(basis_bytes));
        HIP_TRY(hipMemsetAsync(M->gm_basis.p, 0, M->gm_basis.bytes, s));
    }
    HIP_TRY(M->gm_state.alloc((size_t)B * sizeof(rs::GmState)));
    HIP_TRY(M->gm_part.alloc((size_t)B * rs::gm_part_stride() * sizeof(double)));
    if (!M->gm_vpart.p) {
        HIP_TRY(M->gm_vpart.alloc(M->gm_vpart_bytes()));
        rs::launch_flow_mark(M->gm_vpart.p, M->gm_vpart_bytes(), s);
        HIP_TRY(hipGetLastError());
    }
    rs::GmWork g{M->gm_basis.as<double>(), colstride, k.vstride, M->gm_part.as<double>(), rs::gm_part_stride(),
                 k.tickets, (uint32_t)k.ticket_stride, M->spin_limit, M->gm_vpart.as<double>(), M->gm_state.as<rs::GmState>(),
                 k.st};
    const size_t m = 3 * (size_t)M->n * B;
    const double *bd = nullptr;
    st = stage_in(b, mem, M->bstage, m, s, &bd);
    if (st != RS_OK) return st;
    double *xd = x;
    if (mem != RS_MEM_DEVICE) {
        HIP_TRY(M->xstage.alloc(m * sizeof(double)));
        xd = M->xstage.as<double>();
    }
    st = solve_events(M, s);
    if (st != RS_OK) return st;
    {
        // r = rhat = P b, x = 0, ||b||, the initial tests; the first cycle
        // starts from v_0 = r / ||b||
        ProfScope ps(PC_VEC, s, (double)B * 152 * M->n);
        rs::launch_setup(M->an->dev, bd, M->bad.as<int32_t>(), reduction, max_iter, k, B, flow.on, s);
    }
    rs::launch_gm_init(g, B, s);
    rs::launch_gm_normalise(g, k.r, 0, 0, M->n, B, s);
    HIP_TRY(hipGetLastError());
    auto poll = [&](bool &any_run, bool &all_done) -> int {
        HIP_TRY(hipMemcpyAsync(M->h_state, k.st, B * sizeof(SysState), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        any_run = false;
        all_done = true;
        for (int i = 0; i < B; ++i) {
            any_run |= M->h_state[i].phase == rs::PH_RUN;
            all_done &= M->h_state[i].phase == rs::PH_DONE;
        }
        return RS_OK;
    };
    // x back to the caller's order, the true residual, and the results to the host
    auto finish = [&]() -> int {
        rs::launch_finish(M->an->dev, A->rowptr.as<int32_t>(), A->colidx.as<int32_t>(), A->vals.as<double>(),
                          (size_t)A->nnzb * 9, bd, xd, k, B, M->spmv_variant, M->split(), A->wells(), s);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipEventRecord(M->ev_s1, s));
        HIP_TRY(hipMemcpyAsync(M->h_state, k.st, B * sizeof(SysState), hipMemcpyDeviceToHost, s));
        // only single-launch sweeps and applications touch the counters
        if (M->tile_sweeps || flow.on) HIP_TRY(hipMemcpyAsync(M->h_ctr, k.lctr, 2 * sizeof(rs::SweepCtr), hipMemcpyDeviceToHost, s));
        if (mem != RS_MEM_DEVICE) HIP_TRY(hipMemcpyAsync(x, xd, m * sizeof(double), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        M->apply_queued = false;   // `s` came after it
        return RS_OK;
    };
    auto done_all = [&]() {
        bool all = true;
        for (int i = 0; i < B; ++i) all &= M->h_state[i].phase == rs::PH_DONE;
        return all;
    };
    bool any_run = true, all_done = false, finished = false;
    if (!M->predict) {
        st = poll(any_run, all_done);
        if (st != RS_OK) return st;
    }
    // Every cycle advances each system not yet done by at least one step,
    // so max_iter + 1 cycles always suffice.  With prediction the first
    // poll comes after as many steps as the previous solve needed; a cycle
    // that a poll ends (no system iterating) queues the finishing work with
    // its end, so a solve that stops there costs two host synchronisations.
    long long queued = 0;
    long long next_poll = M->predict ? std::max(M->chunk, M->last_gm_steps) : M->chunk;
    for (int cycle = 0; !all_done && cycle <= max_iter; ++cycle) {
        int cols = 0;
        bool stopped = false;
        for (int j = 0; j < restart; ++j) {
            gm_step_any(M, g, j, flow, s);
            ++queued;
            cols = j + 1;
            if (j + 1 == restart) break;
            if (queued >= next_poll) {
                st = poll(any_run, all_done);
                if (st != RS_OK) return st;
                next_poll = queued + M->chunk;
                if (!any_run) {
                    stopped = true;
                    break;
                }
            }
            ProfScope ps(PC_VEC, s, (double)B * 48 * M->n, true);
            rs::launch_gm_normalise(g, k.t, j + 1, 1, M->n, B, s, ps.start(), ps.stop());
        }
        gm_cycle_end_any(M, g, cols, flow, s);
        HIP_TRY(hipGetLastError());
        if (stopped) {
            st = finish();
            if (st != RS_OK) return st;
            if (done_all()) {
                finished = true;
                break;
            }
            continue;
        }
        st = poll(any_run, all_done);
        if (st != RS_OK) return st;
    }
    if (!finished) {
        st = finish();
        if (st != RS_OK) return st;
    }
    if ((st = solve_waits(M, M->tile_sweeps || flow.on, s)) != RS_OK) return st;
    const double solve_ms = elapsed_ms(M->ev_s0, M->ev_s1);
    int worst = RS_OK, needed = 1;
    for (int i = 0; i < B; ++i) {
        const SysState &S = M->h_state[i];
        if (info) info[i] = solve_info{S.status, S.half_steps, S.r0norm, S.last_norm, S.true_res, factor_time(M), solve_ms};
        if (status_rank(S.status) > status_rank(worst)) worst = S.status;
        needed = std::max(needed, S.half_steps);
    }
    if (worst == RS_OK) M->last_gm_steps = std::min(needed, kPredictMax);
    if (worst == RS_HIP_ERROR) factor_message(worst);
    return worst;
}

int rsolve_profile_enable(int32_t mask) {
    prof_flush();
    g_prof.mask = mask;
    for (int c = 0; c < PC_COUNT; ++c) {
        g_prof.ms[c] = 0.0;
        g_prof.bytes[c] = 0.0;
        g_prof.units[c] = 0;
    }
    return RS_OK;
}

int rsolve_profile_set_mask(int32_t mask) {
    g_prof.mask = mask;
    return RS_OK;
}

int rsolve_profile_get(int32_t cls, double *ms, int64_t *units, double *bytes) {
    if (cls < 0 || cls >= PC_COUNT) return fail(RS_INVALID_ARG, "rsolve_profile_get: unknown class");
    prof_flush();
    if (ms) *ms = g_prof.ms[cls];
    if (units) *units = g_prof.units[cls];
    if (bytes) *bytes = g_prof.bytes[cls];
    return RS_OK;
}

// flow: the handle's iterations run their applications as one launch unless
// the tuner's choice says otherwise (fmt 4; the kernels of earlier formats are gone).
static std::string tune_key(ilu0_t M, bool flow) {
    int dev = 0;
    hipDeviceProp_t prop{};
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) prop.multiProcessorCount = 0;
    std::ostringstream k;
    k << "n=" << M->n << ",nnzb=" << M->nnzb << ",batch=" << M->batch << ",ord=" << M->an->sch.ordering
      << ",prec=" << M->precision << ",nl=" << M->an->sch.nl_levels << ",nu=" << M->an->sch.nu_levels
      << ",m=" << M->an->sch.nnz_m << ",fmt=4,path=" << (flow ? "one" : "many")
      << ",arch=" << prop.gcnArchName << ",cu=" << prop.multiProcessorCount;
    std::string r = k.str();
    for (char &c : r)
        if (c == ' ') c = '_';
    return r;
}

// Largest number of wave partials every consumer workgroup adds itself
// (RS_OPT_REDUCE_SPLIT 2) that the autotuner tries.
constexpr int kConsumerSumMax = 8192;

int ilu0_autotune(ilu0_t M, bcsr_t A, const double *b, int32_t mem, double reduction, int32_t reps, void *stream,
                  rs_tune_result *out) {
    int st = check_pair(M, A);
    if (st != RS_OK) return st;
    if (!b || reps < 1 || !(reduction >= 0.0) || (mem != RS_MEM_HOST && mem != RS_MEM_DEVICE))
        return fail(RS_INVALID_ARG, "ilu0_autotune: bad arguments");
    if (!M->factored) return fail(RS_NOT_FACTORED, "ilu0_autotune: call ilu0_factor first");
    hipStream_t s = (hipStream_t)stream;
    rs_tune_result res{M->spmv_variant, M->sweep_variant, M->tile_sweeps ? 1 : 0, M->sweep_grid, 0.0, 0, 0,
                       M->reduce_split};
    const bool flow = flow_size(M, A->nw > 0, false);
    const std::string key = tune_key(M, flow);
    const char *cache = std::getenv("RSOLVE_TUNE_CACHE");
    if (cache && *cache) {
        std::ifstream in(cache);
        std::string line;
        while (std::getline(in, line)) {
            std::istringstream ls(line);
            std::string k;
            rs_tune_result r{};
            if (ls >> k >> r.spmv_variant >> r.sweep_variant >> r.sweep_tiles >> r.sweep_grid >> r.reduce_split &&
                k == key && r.spmv_variant >= 0 && r.spmv_variant < rs::RV_COUNT && r.sweep_variant >= 0 &&
                r.sweep_variant < rs::RV_COUNT && r.sweep_grid >= 1 && r.reduce_split >= 0 && r.reduce_split <= 2) {
                res = r;
                res.from_cache = 1;
            }
        }
        if (res.from_cache) {
            M->spmv_variant = res.spmv_variant;
            M->sweep_variant = res.sweep_variant;
            M->tile_sweeps = res.sweep_tiles != 0;
            M->sweep_grid = res.sweep_grid;
            M->reduce_split = res.reduce_split;
            if (out) *out = res;
            return RS_OK;
        }
    }
    const size_t m = 3 * (size_t)M->n * M->batch;
    DevBuf bb, xb;
    HIP_TRY(bb.alloc(std::max<size_t>(m, 1) * sizeof(double)));
    HIP_TRY(xb.alloc(std::max<size_t>(m, 1) * sizeof(double)));
    if (m)
        HIP_TRY(hipMemcpyAsync(bb.p, b, m * sizeof(double),
                               mem == RS_MEM_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, s));
    struct Cfg {
        int spmv, sweep, tiles, grid, split;
    };
    auto apply = [&](const Cfg &c) {
        M->spmv_variant = c.spmv;
        M->sweep_variant = c.sweep;
        M->tile_sweeps = c.tiles != 0;
        M->sweep_grid = c.grid;
        M->reduce_split = c.split;
    };
    double best = 1e300;
    Cfg bestc{M->spmv_variant, M->sweep_variant, M->tile_sweeps ? 1 : 0, M->sweep_grid, 0};
    int ncand = 0;
    auto time_cfg = [&](const Cfg &c) -> int {
        apply(c);
        // the first solve of a handle learns how many iterations to queue, the
        // second captures graphs of as many
        int r = 0;
        for (int i = 0; i < 2; ++i) {
            r = bicgstab_solve(M, A, bb.as<double>(), xb.as<double>(), reduction, 200, RS_MEM_DEVICE, stream, nullptr);
            if (r < 0) return r;
        }
        const auto t0 = std::chrono::steady_clock::now();
        for (int i = 0; i < reps; ++i) {
            r = bicgstab_solve(M, A, bb.as<double>(), xb.as<double>(), reduction, 200, RS_MEM_DEVICE, stream, nullptr);
            if (r < 0) return r;
        }
        const double us =
            std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / reps;
        ++ncand;
        if (us < best) {
            best = us;
            bestc = c;
        }
        return RS_OK;
    };
    const int sp0 = M->spmv_variant;
    if (flow) {
        // the sweeps of an iteration are part of one launch, whatever their
        // shape: that is timed on the call that takes it, an application
        int sweep = M->sweep_variant;
        double fastest = 1e300;
        for (int v = 0; v < rs::RV_COUNT; ++v) {
            apply({sp0, v, 0, M->sweep_grid, 0});
            st = ilu0_apply(M, bb.as<double>(), xb.as<double>(), 0, M->batch, RS_MEM_DEVICE, stream);
            if (st != RS_OK) return st;
            HIP_TRY(hipStreamSynchronize(s));
            const auto t0 = std::chrono::steady_clock::now();
            for (int i = 0; i < reps; ++i) {
                st = ilu0_apply(M, bb.as<double>(), xb.as<double>(), 0, M->batch, RS_MEM_DEVICE, stream);
                if (st != RS_OK) return st;
            }
            HIP_TRY(hipStreamSynchronize(s));
            const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count();
            ++ncand;
            if (us < fastest) {
                fastest = us;
                sweep = v;
            }
        }
        st = time_cfg({sp0, sweep, 0, M->sweep_grid, 0});
        if (st != RS_OK) return st;
    }
    for (int v = 0; !flow && v < rs::RV_COUNT; ++v) {
        st = time_cfg({sp0, v, 0, M->sweep_grid, 0});
        if (st != RS_OK) return st;
    }
    for (int g : {64, 128, 256}) {
        st = time_cfg({sp0, bestc.sweep, 1, g, 0});
        if (st != RS_OK) return st;
    }
    const Cfg sweep_best = bestc;
    for (int v = 0; v < rs::RV_COUNT; ++v) {
        // one launch forms the product too: its shape would only group the
        // partial sums
        if (v == sp0 || (flow && sweep_best.tiles == 0)) continue;
        st = time_cfg({v, sweep_best.sweep, sweep_best.tiles, sweep_best.grid, 0});
        if (st != RS_OK) return st;
    }
    {
        // the split reductions with the best configuration; consumers adding
        // the wave partials themselves only while those stay few
        const Cfg c = bestc;
        st = time_cfg({c.spmv, c.sweep, c.tiles, c.grid, 1});
        if (st != RS_OK) return st;
        if (rs::spmv_sums(M->n, rs::variant_waves(c.spmv), 2).count <= kConsumerSumMax) {
            st = time_cfg({c.spmv, c.sweep, c.tiles, c.grid, 2});
            if (st != RS_OK) return st;
        }
    }
    apply(bestc);
    res = rs_tune_result{bestc.spmv, bestc.sweep, bestc.tiles, bestc.grid, best, ncand, 0, bestc.split};
    if (cache && *cache) {
        std::ofstream o(cache, std::ios::app);
        o << key << " " << res.spmv_variant << " " << res.sweep_variant << " " << res.sweep_tiles << " "
          << res.sweep_grid << " " << res.reduce_split << " " << res.us_per_solve << "\n";
    }
    if (out) *out = res;
    return RS_OK;
}

int ilu0_destroy(ilu0_t M) {
    delete M;
    return RS_OK;
}

}  // extern "C"
