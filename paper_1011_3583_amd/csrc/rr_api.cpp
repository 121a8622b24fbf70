// rr_api.cpp -- the extern "C" entry points of librr (see include/rr.h).
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "rr_internal.hpp"
#include "rr_kernels.hpp"
#include "rr_plan.hpp"

namespace rr {

static thread_local std::string g_last_error;

int log_level() {
    static const int level = [] {
        const char* v = std::getenv("RR_LOG");
        return v ? std::max(0, std::min(3, std::atoi(v))) : 0;
    }();
    return level;
}

void log_line(int level, const std::string& msg) {
    if (log_level() < level) return;
    static std::mutex mu;   // whole lines from concurrent callers
    std::lock_guard<std::mutex> lk(mu);
    std::fprintf(stderr, "[rr] %s\n", msg.c_str());
}

rr_status fail(rr_status s, const std::string& why) {
    g_last_error = why;
    if (log_level() >= 1) log_line(1, std::string("error ") + rr_status_string(s) + ": " + why);
    return s;
}

void ensure_tune_context() {
    static std::once_flag once;
    std::call_once(once, [] {
        std::string arch = "nodevice";
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            arch = prop.gcnArchName;
        (void)hipGetLastError();   // a host without a GPU leaves an error behind
        int ver = 0;
        if (hipRuntimeGetVersion(&ver) != hipSuccess) ver = HIP_VERSION;
        (void)hipGetLastError();
        tune_set_context(arch + "@hip" + std::to_string(ver));
    });
}

void clear_error() { g_last_error.clear(); }

bool ranges_overlap(uint64_t a, uint64_t na, uint64_t b, uint64_t nb) {
    if (na == 0 || nb == 0) return false;
    return a < b + nb && b < a + na;
}

rr_status hip_fail(hipError_t e, const char* what) {
    char buf[256];
    std::snprintf(buf, sizeof buf, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
    return fail(RR_ERR_HIP, buf);
}

rr_status validate_permute(const void* dst, const void* src, int ndim, const int64_t* dims,
                           const int* perm, int elem_size, Canon* c) {
    std::string why;
    rr_status st = canonicalize(ndim, dims, perm, elem_size, c, &why);
    if (st != RR_OK) return fail(st, why);
    if (c->total_bytes == 0) return RR_OK;
    if (!dst || !src) return fail(RR_ERR_INVALID_ARG, "NULL buffer for a non-empty problem");
    if (ranges_overlap((uint64_t)dst, (uint64_t)c->total_bytes, (uint64_t)src, (uint64_t)c->total_bytes))
        return fail(RR_ERR_ALIAS, "source and destination overlap");
    return RR_OK;
}

}  // namespace rr

using namespace rr;

extern "C" {

rr_status rr_permute(void* dst, const void* src, int ndim, const int64_t* dims, const int* perm,
                     int elem_size, rr_stream_t stream) {
    clear_error();
    Canon c;
    rr_status st = validate_permute(dst, src, ndim, dims, perm, elem_size, &c);
    if (st != RR_OK) return st;
    if (c.total_bytes == 0) return RR_OK;
    Plan p;
    std::string why;
    st = plan_permute((uint64_t)dst, (uint64_t)src, c, current_tile_options(), &p, &why);
    if (st != RR_OK) return fail(st, why);
    if (log_level() >= 2) log_line(2, "rr_permute " + describe(p));
    hipError_t e = launch_plan(p, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "rr_permute launch");
    return RR_OK;
}

static rr_status validate_reorder(const void* dst, const void* src, int ndim, const int64_t* dims,
                                  const int64_t* base, const int64_t* range, int out_ndim, const int* order,
                                  int elem_size, Canon* c, uint64_t* off) {
    std::string why;
    uint64_t span = 0;
    rr_status st = canonicalize_view(ndim, dims, base, range, out_ndim, order, elem_size, c, off, &span, &why);
    if (st != RR_OK) return fail(st, why);
    if (c->total_bytes == 0) return RR_OK;
    if (!dst || !src) return fail(RR_ERR_INVALID_ARG, "NULL buffer for a non-empty problem");
    if (ranges_overlap((uint64_t)dst, (uint64_t)c->total_bytes, (uint64_t)src + *off, span))
        return fail(RR_ERR_ALIAS, "destination overlaps the box read from the source");
    return RR_OK;
}

rr_status rr_reorder(void* dst, const void* src, int ndim, const int64_t* dims, const int64_t* base,
                     const int64_t* range, int out_ndim, const int* order, int elem_size,
                     rr_stream_t stream) {
    clear_error();
    Canon c;
    uint64_t off = 0;
    rr_status st = validate_reorder(dst, src, ndim, dims, base, range, out_ndim, order, elem_size, &c, &off);
    if (st != RR_OK) return st;
    if (c.total_bytes == 0) return RR_OK;
    Plan p;
    std::string why;
    st = plan_permute((uint64_t)dst, (uint64_t)src + off, c, current_tile_options(), &p, &why);
    if (st != RR_OK) return fail(st, why);
    if (log_level() >= 2) log_line(2, std::string("rr_reorder ") + describe(p));
    hipError_t e = launch_plan(p, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "rr_reorder launch");
    return RR_OK;
}

rr_status rr_reorder_describe(const void* dst, const void* src, int ndim, const int64_t* dims,
                              const int64_t* base, const int64_t* range, int out_ndim, const int* order,
                              int elem_size, char* buf, int buflen) {
    clear_error();
    if (!buf || buflen < 1) return fail(RR_ERR_INVALID_ARG, "NULL output buffer");
    Canon c;
    uint64_t off = 0, span = 0;
    std::string why;
    rr_status st = canonicalize_view(ndim, dims, base, range, out_ndim, order, elem_size, &c, &off, &span, &why);
    if (st != RR_OK) return fail(st, why);
    Plan p;
    st = plan_permute((uint64_t)dst, (uint64_t)src + off, c, current_tile_options(), &p, &why);
    if (st != RR_OK) return fail(st, why);
    std::string s = describe(p);
    std::snprintf(buf, (size_t)buflen, "%s", s.c_str());
    return RR_OK;
}

rr_status rr_gather(void* dst, const void* src, int64_t src_count, const int64_t* idx, int64_t count,
                    int elem_size, uint64_t* bad_count, rr_stream_t stream) {
    clear_error();
    if (elem_size < 1 || elem_size > 16) return fail(RR_ERR_INVALID_ARG, "elem_size must be 1..16");
    if (count < 0 || src_count < 0) return fail(RR_ERR_INVALID_ARG, "count and src_count must be >= 0");
    int64_t out_bytes, in_bytes, idx_bytes;
    if (__builtin_mul_overflow(count, (int64_t)elem_size, &out_bytes) ||
        __builtin_mul_overflow(src_count, (int64_t)elem_size, &in_bytes) ||
        __builtin_mul_overflow(count, (int64_t)8, &idx_bytes))
        return fail(RR_ERR_OVERFLOW, "byte count overflows int64");
    if (count == 0) return RR_OK;
    if (!dst || !idx || (!src && src_count > 0)) return fail(RR_ERR_INVALID_ARG, "NULL buffer for a non-empty problem");
    if (ranges_overlap((uint64_t)dst, out_bytes, (uint64_t)src, in_bytes) ||
        ranges_overlap((uint64_t)dst, out_bytes, (uint64_t)idx, idx_bytes) ||
        (bad_count && ranges_overlap((uint64_t)dst, out_bytes, (uint64_t)bad_count, 8)))
        return fail(RR_ERR_ALIAS, "destination overlaps the source, the indices or the counter");
    Plan p;
    plan_gather((uint64_t)dst, (uint64_t)src, (uint64_t)idx, (uint64_t)bad_count, count, src_count, 0, 0, elem_size, &p);
    if (log_level() >= 2) log_line(2, std::string("rr_gather ") + describe(p));
    hipError_t e = launch_plan(p, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "rr_gather launch");
    return RR_OK;
}

rr_status rr_copy_range(void* dst, const void* src, int64_t src_count, int64_t start, int64_t stride,
                        int64_t count, int elem_size, rr_stream_t stream) {
    clear_error();
    if (elem_size < 1 || elem_size > 16) return fail(RR_ERR_INVALID_ARG, "elem_size must be 1..16");
    if (count < 0 || src_count < 0) return fail(RR_ERR_INVALID_ARG, "count and src_count must be >= 0");
    int64_t out_bytes, in_bytes, span, last;
    if (__builtin_mul_overflow(count, (int64_t)elem_size, &out_bytes) ||
        __builtin_mul_overflow(src_count, (int64_t)elem_size, &in_bytes))
        return fail(RR_ERR_OVERFLOW, "byte count overflows int64");
    if (count == 0) return RR_OK;
    if (__builtin_mul_overflow(count - 1, stride, &span) || __builtin_add_overflow(start, span, &last))
        return fail(RR_ERR_OVERFLOW, "range end overflows int64");
    if (start < 0 || start >= src_count || last < 0 || last >= src_count)
        return fail(RR_ERR_INVALID_ARG, "range reads outside the source");
    if (!dst || !src) return fail(RR_ERR_INVALID_ARG, "NULL buffer for a non-empty problem");
    const int64_t lo = std::min(start, last), hi = std::max(start, last);
    if (ranges_overlap((uint64_t)dst, out_bytes, (uint64_t)src + lo * elem_size, (hi - lo + 1) * elem_size))
        return fail(RR_ERR_ALIAS, "destination overlaps the range read");
    Plan p;
    if (stride == 1) plan_copy((uint64_t)dst, (uint64_t)src + start * elem_size, (uint64_t)out_bytes, &p);
    else plan_gather((uint64_t)dst, (uint64_t)src, 0, 0, count, src_count, start, stride, elem_size, &p);
    if (log_level() >= 2) log_line(2, std::string("rr_copy_range ") + describe(p));
    hipError_t e = launch_plan(p, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "rr_copy_range launch");
    return RR_OK;
}

rr_status rr_stencil2d(float* dst, const float* src, int64_t rows, int64_t cols, int radius, int shape,
                       const float* weights, rr_stream_t stream) {
    clear_error();
    if (rows < 0 || cols < 0) return fail(RR_ERR_INVALID_ARG, "rows and cols must be >= 0");
    if (radius < 1 || radius > ST_MAXR) return fail(RR_ERR_INVALID_ARG, "radius must be 1..4");
    if (shape != RR_STENCIL_STAR && shape != RR_STENCIL_BOX) return fail(RR_ERR_INVALID_ARG, "unknown stencil shape");
    if (!weights) return fail(RR_ERR_INVALID_ARG, "NULL weights");
    int64_t n, bytes;
    if (__builtin_mul_overflow(rows, cols, &n) || __builtin_mul_overflow(n, (int64_t)4, &bytes))
        return fail(RR_ERR_OVERFLOW, "grid size overflows int64");
    if (n == 0) return RR_OK;
    if (!dst || !src) return fail(RR_ERR_INVALID_ARG, "NULL grid");
    if (((uint64_t)dst | (uint64_t)src) % 4) return fail(RR_ERR_INVALID_ARG, "grids must be 4-byte aligned");
    if (ranges_overlap((uint64_t)dst, bytes, (uint64_t)src, bytes)) return fail(RR_ERR_ALIAS, "grids overlap");
    StencilArgs a;
    std::memset(&a, 0, sizeof a);
    a.src = (uint64_t)src; a.dst = (uint64_t)dst; a.rows = rows; a.cols = cols;
    a.radius = radius; a.shape = shape;
    const int nw = shape == RR_STENCIL_STAR ? radius + 1 : (2 * radius + 1) * (2 * radius + 1);
    for (int k = 0; k < nw; ++k) a.w[k] = weights[k];
    a.th = stencil_tile_rows(rows, cols);
    const int64_t tx = (cols + ST_TW - 1) / ST_TW, ty = (rows + a.th - 1) / a.th;
    if (tx > 0x7fffffffLL / std::max<int64_t>(ty, 1)) return fail(RR_ERR_UNSUPPORTED, "grid needs too many tiles");
    a.tiles_x = (uint32_t)tx;
    a.ntiles = (uint32_t)(tx * ty);
    hipError_t e = launch_stencil(a, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "rr_stencil2d launch");
    return RR_OK;
}

// Checks an interlace call's arguments and plans it (no launch); *p is left empty
// for count == 0.
static rr_status interlace_plan(void* flat, const void* const* planes, int n, int64_t count, int elem_size,
                                bool de, Plan* p) {
    if (n < 1 || n > RR_MAX_PLANES) return fail(RR_ERR_INVALID_ARG, "n must be 1..RR_MAX_PLANES");
    if (count < 0) return fail(RR_ERR_INVALID_ARG, "count must be >= 0");
    if (elem_size < 1 || elem_size > 16) return fail(RR_ERR_INVALID_ARG, "elem_size must be 1..16");
    if (!planes) return fail(RR_ERR_INVALID_ARG, "plane array is NULL");
    int64_t plane_bytes, total;
    if (__builtin_mul_overflow(count, (int64_t)elem_size, &plane_bytes) ||
        __builtin_mul_overflow(plane_bytes, (int64_t)n, &total))
        return fail(RR_ERR_OVERFLOW, "byte count overflows int64");
    if (count == 0) { p->kind = K_EMPTY; p->grid = 0; return RR_OK; }
    if (!flat) return fail(RR_ERR_INVALID_ARG, "NULL joined buffer");
    uint64_t pl[RR_MAX_PLANES];
    for (int c = 0; c < n; ++c) {
        if (!planes[c]) return fail(RR_ERR_INVALID_ARG, "NULL plane pointer");
        pl[c] = (uint64_t)planes[c];
        if (ranges_overlap(pl[c], plane_bytes, (uint64_t)flat, total))
            return fail(RR_ERR_ALIAS, "a plane overlaps the joined buffer");
    }
    if (de)
        for (int c = 0; c < n; ++c)
            for (int c2 = c + 1; c2 < n; ++c2)
                if (ranges_overlap(pl[c], plane_bytes, pl[c2], plane_bytes))
                    return fail(RR_ERR_ALIAS, "output planes overlap");
    std::string why;
    rr_status st = plan_interlace((uint64_t)flat, pl, n, count, elem_size, de, current_tile_options(), p, &why);
    if (st != RR_OK) return fail(st, why);
    return RR_OK;
}

static rr_status interlace_common(void* flat, const void* const* planes, int n, int64_t count,
                                  int elem_size, rr_stream_t stream, bool de) {
    clear_error();
    Plan p;
    rr_status st = interlace_plan(flat, planes, n, count, elem_size, de, &p);
    if (st != RR_OK || p.kind == K_EMPTY) return st;
    if (log_level() >= 2) log_line(2, std::string("interlace_common ") + describe(p));
    hipError_t e = launch_plan(p, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, de ? "rr_deinterlace launch" : "rr_interlace launch");
    return RR_OK;
}

rr_status rr_interlace(void* dst, const void* const* srcs, int n, int64_t count, int elem_size,
                       rr_stream_t stream) {
    return interlace_common(dst, srcs, n, count, elem_size, stream, false);
}

rr_status rr_deinterlace(void* const* dsts, const void* src, int n, int64_t count, int elem_size,
                         rr_stream_t stream) {
    return interlace_common(const_cast<void*>(src), (const void* const*)dsts, n, count, elem_size,
                            stream, true);
}

rr_status rr_interlace_describe(const void* flat, const void* const* planes, int n, int64_t count,
                                int elem_size, int de, char* buf, int buflen) {
    clear_error();
    if (!buf || buflen < 1) return fail(RR_ERR_INVALID_ARG, "NULL output buffer");
    Plan p;
    rr_status st = interlace_plan(const_cast<void*>(flat), planes, n, count, elem_size, de != 0, &p);
    if (st != RR_OK) return st;
    std::snprintf(buf, (size_t)buflen, "%s", describe(p).c_str());
    return RR_OK;
}

rr_status rr_order_to_perm(int ndim, const int* paper_order, int* perm_out) {
    clear_error();
    if (ndim < 1 || ndim > RR_MAX_DIMS || !paper_order || !perm_out)
        return fail(RR_ERR_INVALID_ARG, "bad ndim or NULL array");
    bool seen[RR_MAX_DIMS] = {};
    for (int k = 0; k < ndim; ++k) {
        int o = paper_order[k];
        if (o < 0 || o >= ndim || seen[o]) return fail(RR_ERR_INVALID_ARG, "order is not a permutation");
        seen[o] = true;
    }
    for (int j = 0; j < ndim; ++j) perm_out[j] = ndim - 1 - paper_order[ndim - 1 - j];
    return RR_OK;
}

rr_status rr_plan_describe(const void* dst, const void* src, int ndim, const int64_t* dims,
                           const int* perm, int elem_size, char* buf, int buflen) {
    clear_error();
    if (!buf || buflen < 1) return fail(RR_ERR_INVALID_ARG, "NULL output buffer");
    Canon c;
    std::string why;
    rr_status st = canonicalize(ndim, dims, perm, elem_size, &c, &why);
    if (st != RR_OK) return fail(st, why);
    Plan p;
    st = plan_permute((uint64_t)dst, (uint64_t)src, c, current_tile_options(), &p, &why);
    if (st != RR_OK) return fail(st, why);
    std::string s = describe(p);
    std::snprintf(buf, (size_t)buflen, "%s", s.c_str());
    return RR_OK;
}

rr_status rr_set_tile_override(int in_row_bytes, int out_row_bytes, int flags) {
    clear_error();
    if (in_row_bytes < 0 || out_row_bytes < 0 || in_row_bytes > 4096 || out_row_bytes > 4096)
        return fail(RR_ERR_INVALID_ARG, "row bytes must be 0..4096");
    const int max_g = (flags >> 8) & 0xff;
    if (!valid_max_g(max_g)) return fail(RR_ERR_INVALID_ARG, "micro-tile cap must be 0, 1, 2, 4, 8 or 16");
    const int tile_kib = (flags >> 16) & 0xff;
    if (!valid_tile_kib(tile_kib)) return fail(RR_ERR_INVALID_ARG, "tile size must be 0 or 4..64 KiB");
    if ((flags & RR_TILE_XCD) && (flags & RR_TILE_NO_XCD))
        return fail(RR_ERR_INVALID_ARG, "RR_TILE_XCD and RR_TILE_NO_XCD together");
    if ((flags & RR_TILE_FILL) && (flags & RR_TILE_NO_FILL))
        return fail(RR_ERR_INVALID_ARG, "RR_TILE_FILL and RR_TILE_NO_FILL together");
    if ((flags & RR_TILE_DIAG) && (flags & RR_TILE_NO_DIAG))
        return fail(RR_ERR_INVALID_ARG, "RR_TILE_DIAG and RR_TILE_NO_DIAG together");
    const int cache = ((flags >> 24) & 0x7) - 1;   // bits 24..26; 27, 28: fill flags; 29: weave; 30: no diag
    if (cache > 3) return fail(RR_ERR_INVALID_ARG, "cache policy must be 0..3");
    TileOptions o;
    o.max_g = max_g;
    o.tile_kib = tile_kib;
    o.xcd = (flags & RR_TILE_XCD) ? 1 : (flags & RR_TILE_NO_XCD) ? 0 : -1;
    o.cache = cache;
    o.diag = (flags & RR_TILE_DIAG) ? 1 : (flags & RR_TILE_NO_DIAG) ? 0 : -1;
    o.fill = (flags & RR_TILE_FILL) ? 1 : (flags & RR_TILE_NO_FILL) ? 0 : -1;
    o.weave = (flags & RR_TILE_NO_WEAVE) ? 0 : 1;
    o.umt = (flags & RR_TILE_UMT_ALWAYS) ? 2 : (flags & RR_TILE_UMT) ? 1 : 0;
    o.in_row_bytes = in_row_bytes;
    o.out_row_bytes = out_row_bytes;
    o.order_out = (flags & RR_TILE_ORDER_IN) ? 0 : (flags & RR_TILE_ORDER_OUT) ? 1 : -1;
    o.force_ragged = (flags & RR_TILE_FORCE_RAGGED) ? 1 : 0;
    set_tile_override(o);
    return RR_OK;
}

rr_status rr_tune_permute(void* dst, const void* src, int ndim, const int64_t* dims, const int* perm,
                          int elem_size, rr_stream_t stream, double* best_us, double* default_us) {
    clear_error();
    ensure_tune_context();
    Canon c;
    rr_status st = validate_permute(dst, src, ndim, dims, perm, elem_size, &c);
    if (st != RR_OK) return st;
    if (best_us) *best_us = 0;
    if (default_us) *default_us = 0;
    if (c.total_bytes == 0 || c.rank == 0 || c.elem_bytes >= RUN_MIN_BYTES) return RR_OK;
    // row targets, traversal order, micro-tile cap, tile size (KiB), XCD ranges,
    // unaligned micro-tiles, cache policy, diagonal order, odd-extent refit (the
    // first candidate is the built-in plan); candidates that plan to the same launch
    // as an earlier one are skipped
    // (diag: the first candidate takes the built-in choice; the others the plain
    // order unless they say otherwise, so the search covers both orders where the
    // built-in choice is diagonal)
    struct Cand { int in_rb, out_rb, order, max_g, kib, xcd = -1, umt = 0, cache = -1, diag = 0, fill = -1; };
    static const Cand cands[] = {
        {0, 0, -1, 0, 0, -1, 0, -1, -1}, {0, 0, 1, 0, 0},        {0, 0, 0, 0, 0},        {0, 0, -1, 0, 64},
        {0, 0, 1, 0, 32},      {128, 256, -1, 0, 64},  {256, 128, -1, 0, 64},  {256, 512, -1, 0, 64},
        {512, 256, -1, 0, 64}, {512, 512, -1, 0, 64},  {1024, 256, -1, 0, 64}, {256, 1024, -1, 0, 64},
        {1024, 1024, -1, 0, 64}, {2048, 512, -1, 0, 64}, {512, 2048, -1, 0, 64}, {256, 512, 1, 0, 64},
        {512, 256, 1, 0, 64},  {256, 128, 1, 0, 64},   {128, 512, 0, 0, 64},   {512, 512, 1, 0, 32},
        {0, 0, -1, 16, 64},    {0, 0, 1, 16, 64},      {512, 512, -1, 16, 64}, {0, 0, -1, 8, 0},
        {0, 0, 1, 8, 0},       {128, 128, -1, 8, 0},   {128, 128, 1, 8, 0},    {256, 128, -1, 8, 0},
        {0, 0, -1, 4, 0},      {0, 0, 1, 4, 0},        {128, 128, -1, 4, 0},   {64, 128, 1, 4, 0},
        {128, 64, 1, 4, 0},    {64, 256, -1, 4, 0},    {64, 256, -1, 16, 0},   {64, 256, -1, 16, 32},
        {128, 128, -1, 16, 0}, {0, 0, -1, 0, 0, 1},    {0, 0, 1, 0, 0, 1},     {0, 0, 0, 0, 0, 1},
        {0, 0, -1, 0, 64, 1},  {512, 512, -1, 16, 64, 1}, {0, 0, -1, 0, 0, 0, 1}, {0, 0, 1, 0, 0, 0, 1},
        {0, 0, 0, 0, 0, 0, 1}, {512, 512, -1, 0, 64, 0, 1},
        {0, 0, -1, 0, 0, 0, 0, 0}, {0, 0, -1, 0, 0, 0, 0, 1}, {0, 0, -1, 0, 0, 1, 0, 1},
        {0, 0, -1, 0, 0, 0, 0, 2}, {0, 0, -1, 0, 0, 1, 0, 2}, {0, 0, -1, 0, 0, 1, 0, 3},
        {0, 0, 1, 0, 0, 1, 0, 1},  {0, 0, 0, 0, 0, 1, 0, 2}, {512, 512, -1, 0, 64, 1, 0, 1},
        {0, 0, -1, 0, 0, -1, 0, -1, 1}, {0, 0, 0, 0, 0, -1, 0, -1, 1}, {0, 0, -1, 0, 64, -1, 0, -1, 1},
        {1024, 256, 1, 0, 0, -1, 0, -1, 1}, {256, 1024, 1, 0, 0, -1, 0, -1, 1}, {512, 512, 0, 0, 0, -1, 0, -1, 1},
        {0, 0, -1, 0, 0, -1, 0, -1, 0, 0}, {0, 0, 1, 0, 0, -1, 0, -1, 0, 0}, {0, 0, 0, 0, 0, -1, 0, -1, 0, 0},
        {512, 512, -1, 0, 64, -1, 0, -1, 0, 0}, {0, 0, -1, 0, 0, -1, 0, -1, 0}};
    hipStream_t hs = (hipStream_t)stream;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return fail(RR_ERR_HIP, "hipEventCreate");
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return fail(RR_ERR_HIP, "hipEventCreate"); }
    // Every timed run starts from caches that hold none of the problem (a write of
    // twice the Infinity Cache's 256 MB): re-running one problem back to back
    // would otherwise find a small input still cached and favour cached loads.
    constexpr size_t FLUSH_BYTES = size_t(512) << 20;
    void* flush = nullptr;
    if (hipMalloc(&flush, FLUSH_BYTES) != hipSuccess) { flush = nullptr; (void)hipGetLastError(); }
    double best = 1e300, def = 0;
    TileOptions bestopt;
    std::vector<std::string> seen;
    for (const Cand& cd : cands) {
        TileOptions o;
        o.in_row_bytes = cd.in_rb;
        o.out_row_bytes = cd.out_rb;
        o.order_out = cd.order;
        o.max_g = cd.max_g;
        o.tile_kib = cd.kib;
        o.xcd = cd.xcd;
        o.umt = cd.umt;
        o.cache = cd.cache;
        o.diag = cd.diag;
        o.fill = cd.fill;
        Plan p;
        std::string why;
        if (plan_permute((uint64_t)dst, (uint64_t)src, c, o, &p, &why) != RR_OK) continue;
        // skip candidates that plan to a launch already timed
        const std::string sig = describe(p);
        if (std::find(seen.begin(), seen.end(), sig) != seen.end()) continue;
        seen.push_back(sig);
        std::vector<float> ts;
        for (int r = 0; r < 4 && st == RR_OK; ++r) {
            if (flush) (void)hipMemsetAsync(flush, r & 0xff, FLUSH_BYTES, hs);
            (void)hipEventRecord(e0, hs);
            hipError_t e = launch_plan(p, hs);
            (void)hipEventRecord(e1, hs);
            if (e != hipSuccess) { st = hip_fail(e, "tuning launch"); break; }
            if ((e = hipEventSynchronize(e1)) != hipSuccess) { st = hip_fail(e, "tuning sync"); break; }
            float ms = 0;
            (void)hipEventElapsedTime(&ms, e0, e1);
            if (r > 0) ts.push_back(ms);
        }
        if (st != RR_OK) break;
        std::sort(ts.begin(), ts.end());
        const double us = ts[ts.size() / 2] * 1e3;
        if (&cd == &cands[0]) def = us;
        if (us < best) { best = us; bestopt = o; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (flush) {
        (void)hipStreamSynchronize(hs);
        (void)hipFree(flush);
    }
    if (st != RR_OK) return st;
    tune_store(tune_key(c, (uint64_t)dst, (uint64_t)src), bestopt);
    if (best_us) *best_us = best;
    if (default_us) *default_us = def;
    return RR_OK;
}

rr_status rr_tune_save(const char* path) {
    clear_error();
    if (!path) return fail(RR_ERR_INVALID_ARG, "NULL path");
    FILE* f = std::fopen(path, "w");
    if (!f) return fail(RR_ERR_INVALID_ARG, std::string("cannot write ") + path);
    ensure_tune_context();
    const std::string s = tune_dump();
    std::fwrite(s.data(), 1, s.size(), f);
    std::fclose(f);
    return RR_OK;
}

rr_status rr_tune_load(const char* path) {
    clear_error();
    if (!path) return fail(RR_ERR_INVALID_ARG, "NULL path");
    FILE* f = std::fopen(path, "r");
    if (!f) return fail(RR_ERR_INVALID_ARG, std::string("cannot read ") + path);
    std::string s;
    char buf[4096];
    size_t n;
    while ((n = std::fread(buf, 1, sizeof buf, f)) > 0) s.append(buf, n);
    std::fclose(f);
    ensure_tune_context();
    int skipped = 0;
    if (tune_parse(s, &skipped) < 0) return fail(RR_ERR_INVALID_ARG, "malformed tuning file");
    if (skipped && log_level() >= 1)
        log_line(1, std::string(path) + ": " + std::to_string(skipped) + " tuned shapes of another device or HIP "
                    "version skipped (this process: " + tune_context() + ")");
    return RR_OK;
}

rr_status rr_tune_context(char* buf, int buflen) {
    clear_error();
    if (!buf || buflen < 1) return fail(RR_ERR_INVALID_ARG, "NULL buffer");
    ensure_tune_context();
    const std::string c = tune_context();
    if ((int)c.size() + 1 > buflen) return fail(RR_ERR_INVALID_ARG, "buffer too short");
    std::memcpy(buf, c.c_str(), c.size() + 1);
    return RR_OK;
}

rr_status rr_tune_clear(void) {
    clear_error();
    tune_clear();
    return RR_OK;
}

const char* rr_status_string(rr_status s) {
    switch (s) {
        case RR_OK: return "RR_OK";
        case RR_ERR_INVALID_ARG: return "RR_ERR_INVALID_ARG";
        case RR_ERR_OVERFLOW: return "RR_ERR_OVERFLOW";
        case RR_ERR_ALIAS: return "RR_ERR_ALIAS";
        case RR_ERR_UNSUPPORTED: return "RR_ERR_UNSUPPORTED";
        case RR_ERR_NO_MEMORY: return "RR_ERR_NO_MEMORY";
        case RR_ERR_BUSY: return "RR_ERR_BUSY";
        case RR_ERR_NOT_READY: return "RR_ERR_NOT_READY";
        case RR_ERR_HIP: return "RR_ERR_HIP";
    }
    return "RR_ERR_UNKNOWN";
}

const char* rr_last_error(void) { return g_last_error.c_str(); }

const char* rr_version(void) { return "librr 0.1 (gfx950)"; }

}  // extern "C"
