// Host side of the C ABI (include/sivf.h): context and workspace management,
// input validation, and the sequencing of the assignment step (Alg. 4),
// update step (Alg. 5) and Lloyd driver (Alg. 1) on one HIP stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <new>
#include <vector>

#include "internal.h"
#include "soft.h"
#include "sort.h"

using namespace sivf;

namespace {

sivf_status fail(sivf_ctx* ctx, sivf_status st, const char* fmt, ...) {
    if (ctx) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof(buf), fmt, ap);
        va_end(ap);
        ctx->err = buf;
    }
    return st;
}

#define HIPCHK(ctx, expr)                                                                          \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return fail((ctx), SIVF_E_HIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                        __FILE__, __LINE__);                                                       \
    } while (0)

#define STCHK(expr)                      \
    do {                                 \
        sivf_status s_ = (expr);         \
        if (s_ != SIVF_OK) return s_;    \
    } while (0)

struct DevGuard {
    int prev = -1;
    explicit DevGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DevGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

bool cap_ok(sivf_ctx* ctx, size_t more) {
    return ctx->opt.workspace_cap_bytes == 0 || ctx->bytes_held + more <= ctx->opt.workspace_cap_bytes;
}

void dev_free(sivf_ctx* ctx, void* p, size_t bytes, size_t* account) {
    if (!p) return;
    if (bytes == 0) bytes = 8;
    (void)hipFree(p);
    ctx->bytes_held -= std::min(ctx->bytes_held, bytes);
    if (account) *account -= std::min(*account, bytes);
}

// Frees what the ctx holds for faster forms only: its optional buffers, and the
// sliced rows of the file that is being updated.  None of it is in use then: a
// call asks for what it cannot do without first, and the stream is waited for.
// Returns whether there was anything.
bool give_back(sivf_ctx* ctx) {
    sivf_ivf* f = ctx->updating;
    bool any = f && f->sval;
    for (const auto& kv : ctx->ws) any = any || kv.second.optional;
    if (!any || hipStreamSynchronize(ctx->stream) != hipSuccess) return false;
    for (auto it = ctx->ws.begin(); it != ctx->ws.end();) {
        if (!it->second.optional) {
            ++it;
            continue;
        }
        dev_free(ctx, it->second.p, it->second.bytes, nullptr);
        it = ctx->ws.erase(it);
    }
    if (f && f->sval) {
        dev_free(ctx, f->sval, (size_t)f->scap * 4, &f->bytes);
        f->sval = nullptr;
        f->scap = f->srows = 0;
    }
    return true;
}

sivf_status dev_alloc(sivf_ctx* ctx, void** p, size_t bytes, size_t* account) {
    *p = nullptr;
    if (bytes == 0) bytes = 8;
    if (!cap_ok(ctx, bytes) && !(give_back(ctx) && cap_ok(ctx, bytes)))
        return fail(ctx, SIVF_E_NOMEM, "workspace cap of %zu bytes exceeded (%zu held, %zu requested)",
                    ctx->opt.workspace_cap_bytes, ctx->bytes_held, bytes);
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (give_back(ctx)) e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return fail(ctx, SIVF_E_NOMEM, "hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
    }
    ctx->bytes_held += bytes;
    if (account) *account += bytes;
    return SIVF_OK;
}

// Memory for a faster form that a call can do without: at most half of what is
// free, so that the caller's next allocations find room, and no error if there
// is none.
bool optional_alloc(sivf_ctx* ctx, void** p, size_t bytes, size_t* account) {
    *p = nullptr;
    size_t room = 0, all = 0;
    if (!cap_ok(ctx, bytes) || hipMemGetInfo(&room, &all) != hipSuccess || bytes > room / 2 ||
        hipMalloc(p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return false;
    }
    ctx->bytes_held += bytes;
    if (account) *account += bytes;
    return true;
}

// Grow-only named workspace buffer owned by the ctx.
template <typename T>
sivf_status ws(sivf_ctx* ctx, const char* name, int64_t elems, T** out) {
    size_t bytes = (size_t)std::max<int64_t>(elems, 1) * sizeof(T);
    auto it = ctx->ws.find(name);
    if (it != ctx->ws.end() && it->second.bytes >= bytes) {
        *out = (T*)it->second.p;
        return SIVF_OK;
    }
    if (it != ctx->ws.end()) {
        HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
        dev_free(ctx, it->second.p, it->second.bytes, nullptr);
        ctx->ws.erase(it);
    }
    size_t grow = bytes + bytes / 8;
    void* p = nullptr;
    STCHK(dev_alloc(ctx, &p, grow, nullptr));
    ctx->ws[name] = {p, grow, false};
    *out = (T*)p;
    return SIVF_OK;
}

// Named buffers of a faster form: all of them, or none (the ctx then holds none
// of them).  To be asked for after everything the call cannot do without; later
// calls give them back where they need the room.
struct Optional {
    const char* name;
    size_t bytes;
    void** p;
};

bool ws_optional(sivf_ctx* ctx, std::initializer_list<Optional> list) {
    auto granted = [](size_t bytes) { return bytes + bytes / 8 + 8; };
    size_t more = 0, room = 0, all = 0;
    for (const Optional& q : list) {
        auto it = ctx->ws.find(q.name);
        if (it != ctx->ws.end() && it->second.bytes >= q.bytes) *q.p = it->second.p;
        else more += granted(q.bytes);
    }
    if (more == 0) return true;
    bool ok = hipStreamSynchronize(ctx->stream) == hipSuccess;
    auto drop = [&](bool whole) {
        for (const Optional& q : list) {
            auto it = ctx->ws.find(q.name);
            if (it == ctx->ws.end() || (!whole && it->second.bytes >= q.bytes)) continue;
            dev_free(ctx, it->second.p, it->second.bytes, nullptr);
            ctx->ws.erase(it);
        }
    };
    if (ok) drop(false);
    // together at most half of what is free (each is then at most half of what is left)
    ok = ok && hipMemGetInfo(&room, &all) == hipSuccess && more <= room / 2;
    for (const Optional& q : list) {
        if (!ok) break;
        if (ctx->ws.count(q.name)) continue;
        ok = optional_alloc(ctx, q.p, granted(q.bytes), nullptr);
        if (ok) ctx->ws[q.name] = {*q.p, granted(q.bytes), true};
    }
    if (!ok) {
        (void)hipGetLastError();
        drop(true);
        for (const Optional& q : list) *q.p = nullptr;
    }
    return ok;
}

// Frees the named buffers whose names begin so.
void ws_drop(sivf_ctx* ctx, std::initializer_list<const char*> prefixes) {
    if (hipStreamSynchronize(ctx->stream) != hipSuccess) return;
    for (auto it = ctx->ws.begin(); it != ctx->ws.end();) {
        bool drop = false;
        for (const char* q : prefixes) drop = drop || it->first.compare(0, strlen(q), q) == 0;
        if (drop) dev_free(ctx, it->second.p, it->second.bytes, nullptr);
        it = drop ? ctx->ws.erase(it) : std::next(it);
    }
}

// The same, cleared when it is allocated (all of it: a later, larger request
// may fit what was granted).
template <typename T>
sivf_status ws_zeroed(sivf_ctx* ctx, const char* name, int64_t elems, T** out) {
    static_assert(sizeof(T) == 8, "cleared by 8-byte words");
    auto it = ctx->ws.find(name);
    void* before = it == ctx->ws.end() ? nullptr : it->second.p;
    const size_t size = it == ctx->ws.end() ? 0 : it->second.bytes;
    STCHK(ws(ctx, name, elems, out));
    const auto& got = ctx->ws[name];
    if (got.p != before || got.bytes != size)
        HIPCHK(ctx, fill_u64((unsigned long long*)got.p, 0ull, (int64_t)(got.bytes / 8), ctx->stream));
    return SIVF_OK;
}

// Buffers of a sort of n entries ("<name>_..."); val: with values.
template <typename V>
sivf_status sort_ws(sivf_ctx* ctx, const std::string& name, int64_t n, bool val, SortWs<V>* w) {
    for (int b = 0; b < 2; ++b) {
        const std::string i = std::to_string(b);
        STCHK(ws(ctx, (name + "_key" + i).c_str(), n, &w->key[b]));
        STCHK(ws(ctx, (name + "_row" + i).c_str(), n, &w->row[b]));
        if (val) STCHK(ws(ctx, (name + "_val" + i).c_str(), n, &w->val[b]));
    }
    const int64_t table = sort_table_elems(n);
    STCHK(ws(ctx, (name + "_count").c_str(), table, &w->count));
    STCHK(ws(ctx, (name + "_start").c_str(), table, &w->start));
    return ws(ctx, (name + "_scan").c_str(), scan_ws_elems(table) + 8, &w->scan_ws);
}

// Workspace of one call, handed out buffer by buffer: the ctx's grow-only
// named buffers (kCtx), consecutive 256-byte aligned pieces of a fixed device
// block that is never allocated or freed here (kFixed), or no memory at all,
// only the byte count such a block needs for the same requests (kMeasure).
struct Work {
    enum Mode { kCtx, kFixed, kMeasure };
    sivf_ctx* ctx;
    Mode mode = kCtx;
    char* base = nullptr;
    size_t cap = 0, used = 0;

    template <typename T>
    sivf_status get(const char* name, int64_t elems, T** out) {
        if (mode == kCtx) return ws(ctx, name, elems, out);
        const size_t bytes = (size_t)std::max<int64_t>(elems, 1) * sizeof(T);
        const size_t at = (used + 255) & ~(size_t)255;
        if (mode == kFixed && at + bytes > cap)
            return fail(ctx, SIVF_E_UNSUPPORTED, "workspace '%s' does not fit the %zu-byte scratch block", name, cap);
        *out = (T*)(base + at);   // kMeasure: an offset, never dereferenced
        used = at + bytes;
        return SIVF_OK;
    }
};

// ------------------------------------------------------------ fixed scratch
// The workspace of sivf_assign_noalloc: one block per device, part of the
// library's device code, so the loader provides it when the library is first
// used on a device and it stays until the process ends.  Host code never
// names the array itself (that is a host-side stand-in, not a device
// address): it uses the address hipGetSymbolAddress reports for each device,
// taken once per device with that device current, when a ctx is created.
constexpr size_t kScratchBytes = 64ull << 20;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// device must be current
hipError_t scratch_setup(int device) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = p;
    return hipSuccess;
}

void* scratch_of(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_ptr[device];
}

sivf_status check_csr_args(sivf_ctx* ctx, const sivf_csr* X, const char* what) {
    if (!X) return fail(ctx, SIVF_E_INVALID, "%s is NULL", what);
    if (X->n_rows < 0 || X->n_cols < 1 || X->nnz < 0)
        return fail(ctx, SIVF_E_SHAPE, "%s: bad sizes n_rows=%lld n_cols=%lld nnz=%lld", what, (long long)X->n_rows,
                    (long long)X->n_cols, (long long)X->nnz);
    if (X->n_cols > INT32_MAX) return fail(ctx, SIVF_E_SHAPE, "%s: n_cols exceeds int32", what);
    if (!X->row_ptr || (X->nnz > 0 && (!X->col || !X->val)))
        return fail(ctx, SIVF_E_INVALID, "%s: NULL array", what);
    if (X->val_dtype != SIVF_F32 && X->val_dtype != SIVF_F64)
        return fail(ctx, SIVF_E_INVALID, "%s: values must be SIVF_F32 or SIVF_F64", what);
    return SIVF_OK;
}

// Assignments to check along with a matrix: every a[i] must lie in [0, k)
// before it is used as an index on the device.
struct Ids {
    const int32_t* a;
    int64_t n;
    int32_t k;
    const char* what;
};

// Run the device check on M and the id arrays (at most two) and report what it
// found; *nonneg = no value of M is negative.  flags: 8 words.  Waits for the
// stream once.
sivf_status check_csr(sivf_ctx* ctx, const sivf_csr* M, const char* what, unsigned long long* flags, int* nonneg,
                      std::initializer_list<Ids> ids = {}) {
    const int f64 = M->val_dtype == SIVF_F64;
    unsigned long long* h = (unsigned long long*)ctx->pin;
    HIPCHK(ctx, validate_csr(M->row_ptr, M->col, M->val, f64, M->n_rows, M->n_cols, M->nnz, flags, ctx->stream));
    int q = 4;
    for (const Ids& i : ids) HIPCHK(ctx, range_check_i32(i.a, i.n, i.k, flags + q++, ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(h, flags, 8 * sizeof(*h), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    *nonneg = h[2] ? 0 : 1;
    if (h[0] == 0 && h[3] == 0) {
        q = 4;
        for (const Ids& i : ids)
            if (h[q++]) return fail(ctx, SIVF_E_RANGE, "%s has a value outside [0, %d)", i.what, i.k);
        return SIVF_OK;
    }
    HIPCHK(ctx, validate_csr_rows(M->row_ptr, M->col, M->val, f64, M->n_rows, M->n_cols, M->nnz, flags, ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(h, flags, 4 * sizeof(*h), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    const unsigned long long row = ~h[1];
    if (h[0] & 1ull) return fail(ctx, SIVF_E_UNSORTED, "%s: row %llu has unsorted/duplicate columns or a decreasing row_ptr", what, row);
    if (h[0] & 8ull) return fail(ctx, SIVF_E_UNSORTED, "%s: row_ptr[0] != 0 or row_ptr[n] != nnz", what);
    if (h[0] & 2ull) return fail(ctx, SIVF_E_RANGE, "%s: row %llu has a column outside [0, %lld)", what, row, (long long)M->n_cols);
    if (h[0] & 4ull) return fail(ctx, SIVF_E_NONFINITE, "%s: row %llu has a non-finite value", what, row);
    return fail(ctx, SIVF_E_UNSORTED, "%s changed while it was being checked", what);
}

// Validate X on the device on every call that reads it.  Nothing is cached:
// X may be edited in place between calls (same pointers, new contents), and
// both the column range (used as an index by the walk) and the sign of the
// values (which selects the certificate's error bound) must hold for the
// contents the kernels will read.  One coalesced pass over the nonzeros.
sivf_status validate(sivf_ctx* ctx, const sivf_csr* X, Csr* out, Work& w, std::initializer_list<Ids> ids = {}) {
    STCHK(check_csr_args(ctx, X, "X"));
    unsigned long long* flags = nullptr;
    STCHK(w.get("vflags", 8, &flags));
    if (X->n_rows == 0) {
        int64_t* rp0 = (int64_t*)ctx->pin;
        HIPCHK(ctx, hipMemcpyAsync(rp0, X->row_ptr, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
        HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
        if (*rp0 != 0 || X->nnz != 0) return fail(ctx, SIVF_E_UNSORTED, "X: empty matrix with row_ptr[0] != 0 or nnz != 0");
    }
    int nonneg = 1;
    STCHK(check_csr(ctx, X, "X", flags, &nonneg, ids));
    out->n = X->n_rows;
    out->d = X->n_cols;
    out->nnz = X->nnz;
    out->rp = X->row_ptr;
    out->col = X->col;
    out->val = X->val;
    out->f64 = X->val_dtype == SIVF_F64;
    out->nonneg = nonneg;
    return SIVF_OK;
}

sivf_status validate(sivf_ctx* ctx, const sivf_csr* X, Csr* out, std::initializer_list<Ids> ids = {}) {
    Work w{ctx};
    return validate(ctx, X, out, w, ids);
}

// The split walk reads the head rows faster than the plain one, but moves a sum
// per object and slot through memory and takes three launches per range and
// tile.  FP32 postings only (BF16 rows are half the bytes, and the plain walk
// reads them faster: 500,000 objects, k = 10,000, 42 against 67 ms), not for
// IVF-CBICP (it walks lists), not with a workspace cap (it needs up to 4 GiB) or
// several tiles per launch.  It reads more rows than the plain walk, down to
// 0.6 of head_density: 2,000,000 objects, k = 10,000, 228 ms at 1.0, 212 at
// 0.6, 210 at 0.4; 1,000,000, k = 1,000, 14.2, 13.4 and 13.6.
constexpr double kSplitDensity = 0.6;

bool split_possible(const sivf_options& o) {
    return o.posting_dtype == SIVF_F32 && o.filter_mode != SIVF_MODE_CBICP && o.workspace_cap_bytes == 0 &&
           o.tiles_per_launch <= 1 && o.head_density > 0.0f;
}

// What it saves and costs per object and centroid grows with the sliced terms
// per object (h): about (h - 38) 0.1 ps, and 0.13 ms a tile are lost.  Plain and
// split, ms: k = 10,000: h = 21 65.1 and 76.8 (1,000,000 objects), 34 8.8 and 9.1
// (100,000), 42 27.3 and 25.6 (300,000), 52 100.6 and 87.5 (1,000,000); k = 4,000,
// 100,000 objects, h = 76 6.4 and 5.4; k = 1,000, h = 84: 16,384 objects 0.37 and
// 0.35, 1,000,000 19.1 and 13.1; k = 300, h = 48, 60,000 0.49 and 0.66, h = 58,
// 400,000 2.10 and 2.04.  Few rows stay in L2 anyway (37 rows, h = 41: 18.2 and
// 18.9; 270 rows, h = 42 27.3 and 25.6).
constexpr int64_t kSplitMinRows = 128;
bool split_pays(double h, int64_t objects, int32_t k, int32_t tiles) {
    return (h - 38.0) * (double)objects * (double)k >= 1e9 * tiles;
}

// ---------------------------------------------------------------- file storage
// Several arrays in one allocation (each 256-byte aligned; an allocation and its
// release cost 20 to 60 us whatever their size: a restart's file took 19 of
// them, 1.4 of its 3.1 ms).
struct Piece {
    void** p;
    size_t bytes;
};

size_t pieces_bytes(std::initializer_list<Piece> list) {
    size_t n = 0;
    for (const Piece& q : list) n += (q.bytes + 255) & ~(size_t)255;
    return n;
}

sivf_status pieces_alloc(sivf_ctx* ctx, std::initializer_list<Piece> list, void** block, size_t* block_bytes,
                         size_t* account) {
    const size_t n = pieces_bytes(list);
    STCHK(dev_alloc(ctx, block, n, account));
    *block_bytes = n;
    char* at = (char*)*block;
    for (const Piece& q : list) {
        *q.p = q.bytes ? at : nullptr;
        at += (q.bytes + 255) & ~(size_t)255;
    }
    return SIVF_OK;
}

sivf_status store_reserve(sivf_ctx* ctx, sivf_ivf* f, Store* st, StoreBlock* b, int64_t cap) {
    if (st->cap >= cap && st->term) return SIVF_OK;
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    dev_free(ctx, b->mem, b->bytes, &f->bytes);
    b->mem = nullptr;
    st->term = nullptr;
    st->val = nullptr;
    st->cap = 0;
    int64_t c = std::max<int64_t>(cap + cap / 8, 64);
    STCHK(pieces_alloc(ctx, {{(void**)&st->val, (size_t)c * sizeof(double)}, {(void**)&st->term, (size_t)c * sizeof(int32_t)}},
                       &b->mem, &b->bytes, &f->bytes));
    st->cap = c;
    return SIVF_OK;
}

sivf_status postings_reserve(sivf_ctx* ctx, sivf_ivf* f, int64_t P) {
    // spare entries: the walk reads postings in aligned groups of 8, which
    // may reach up to 7 entries past the last one
    if (f->pcap >= P + 8 && f->cid) return SIVF_OK;
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    dev_free(ctx, f->postings, f->postings_bytes, &f->bytes);
    f->postings = nullptr;
    f->cid = nullptr;
    f->v32 = nullptr;
    f->v16 = nullptr;
    f->v64 = nullptr;
    f->pcap = 0;
    const int64_t c = std::max<int64_t>(P + P / 8 + 8, 64);
    const bool bf16 = f->pdt == SIVF_BF16;
    STCHK(pieces_alloc(ctx, {{(void**)&f->v64, (size_t)c * 8}, {(void**)&f->v32, bf16 ? 0 : (size_t)c * 4},
                             {(void**)&f->v16, bf16 ? (size_t)c * 2 : 0}, {(void**)&f->cid, (size_t)c * 2}},
                       &f->postings, &f->postings_bytes, &f->bytes));
    f->pcap = c;
    return SIVF_OK;
}

void free_file(sivf_ctx* ctx, sivf_ivf* f) {
    if (!f) return;
    (void)hipStreamSynchronize(ctx->stream);
    for (StoreBlock* b : {&f->cur_mem, &f->nxt_mem}) dev_free(ctx, b->mem, b->bytes, &f->bytes);
    dev_free(ctx, f->postings, f->postings_bytes, &f->bytes);
    dev_free(ctx, f->sval, (size_t)f->scap * 4, &f->bytes);
    dev_free(ctx, f->hval, (size_t)f->hcap * (f->pdt == SIVF_BF16 ? 2 : 4), &f->bytes);
    dev_free(ctx, f->fixed, f->fixed_bytes, &f->bytes);
    delete f;
}

sivf_status new_file(sivf_ctx* ctx, int32_t k, int64_t d, sivf_ivf** out) {
    sivf_ivf* f = new (std::nothrow) sivf_ivf();
    if (!f) return fail(ctx, SIVF_E_NOMEM, "host allocation failed");
    f->k = k;
    f->d = d;
    f->pdt = ctx->opt.posting_dtype;
    f->k_tile = ctx->opt.k_tile;
    // arrays for the most tiles the file may come to have
    choose_tiles(f->k_tile, f->pdt == SIVF_BF16, k, INFINITY, d, INT64_MAX, INFINITY, &f->kt, &f->T);
    f->T_max = f->T;
    const size_t kk = (size_t)k, dd = (size_t)d, dt = (size_t)(d * f->T);
    const size_t hd = ctx->opt.head_density > 0.0f ? dd : 0, sd = split_possible(ctx->opt) ? dd : 0;
    const sivf_status st = pieces_alloc(
        ctx, {{(void**)&f->cur.start, kk * 8}, {(void**)&f->cur.nnz, kk * 8}, {(void**)&f->nxt.start, kk * 8},
              {(void**)&f->nxt.nnz, kk * 8}, {(void**)&f->seg, (dt + 1) * 8}, {(void**)&f->mid, dt * 4},
              {(void**)&f->rec, dt * 16}, {(void**)&f->perm, kk * 4}, {(void**)&f->iperm, kk * 4},
              {(void**)&f->lam, kk}, {(void**)&f->cnorm, kk * 8}, {(void**)&f->head, hd * 4},
              {(void**)&f->meta, kMeta * 8}, {(void**)&f->tlen, sd * 8}, {(void**)&f->srow, sd * 4}},
        &f->fixed, &f->fixed_bytes, &f->bytes);
    if (st != SIVF_OK) {
        free_file(ctx, f);
        return st;
    }
    *out = f;
    return SIVF_OK;
}

// Structure f's current centroids by the flags in f->lam (Alg. 5 second half):
// positions put the moving centroids first, then the file is built by position.
// norms: f->cnorm has yet to be computed (the update fills it).
// postings: an estimate of their entries.  X: objects likely to walk it (nullptr:
// unknown); the split walk's rows are made if it pays for them.  A file built from
// given centroids gets none before its first update (they take 0.17 ms of a 3.0 ms
// restart, and nobody may walk it so).
sivf_status restructure(sivf_ctx* ctx, sivf_ivf* f, bool norms, double postings, const Csr* X) {
    // the tiles follow from the options the file was made with: a ctx with others
    // may update it, and its arrays have room for T_max tiles
    int32_t kt = 0, T = 0;
    const bool bf16 = f->pdt == SIVF_BF16;
    choose_tiles(f->k_tile, bf16, f->k, postings, f->d, 0, 0.0, &kt, &T);
    if (X && X->n > 0) {
        // rows that X will walk as they are, some tiles a launch (the rows and the split
        // walk's share taken to be what the file had so far)
        const double terms = (double)X->nnz / (double)X->n;
        int32_t kt2 = 0, T2 = 0;
        choose_tiles(f->k_tile, bf16, f->k, postings, f->d, f->H, terms, &kt2, &T2);
        const bool split_X = !bf16 && split_possible(ctx->opt) && split_pays(f->sfrac * terms, X->n, f->k, T);
        if (!split_X && ctx->opt.tiles_per_launch < T2) {
            kt = kt2;
            T = T2;
        }
    }
    f->built = false;   // until every array below is whole again
    if (T > f->T_max) return fail(ctx, SIVF_E_HIP, "internal: %d tiles in a file made for %d", T, f->T_max);
    f->kt = kt;
    f->T = T;
    const int64_t W64 = ivf_w64(f->k);
    const int64_t nseg2 = f->d * f->T * 2;
    IvfBuildWs w{};
    STCHK(ws(ctx, "ivf_bm", W64 * f->d, &w.bm));
    STCHK(ws(ctx, "ivf_pre0", W64 * f->d, &w.pre0));
    STCHK(ws(ctx, "ivf_pre1", W64 * f->d, &w.pre1));
    STCHK(ws(ctx, "ivf_cnt", nseg2, &w.cnt));
    STCHK(ws(ctx, "ivf_off", nseg2 + 1, &w.off));
    STCHK(ws(ctx, "scan_ws", scan_ws_elems(nseg2) + 8, &w.scan_ws));
    int64_t *cscan = nullptr, *meta = f->meta;
    int32_t *hterm = nullptr, *sterm = nullptr;
    STCHK(ws(ctx, "ivf_cscan", (int64_t)f->k + 1, &cscan));
    if (f->head) STCHK(ws(ctx, "head_term", f->d, &hterm));
    if (f->srow) STCHK(ws(ctx, "split_term", f->d, &sterm));
    HIPCHK(ctx, ivf_perm(f->lam, f->k, f->cur.nnz, f->perm, f->iperm, cscan, meta, ctx->stream));
    HIPCHK(ctx, ivf_count(f->cur, f->k, f->d, f->kt, f->T, f->iperm, cscan, meta, w, ctx->stream));
    // dense head rows: terms whose lists hold >= ceil(head_density * k) postings;
    // sliced rows: down to kSplitDensity of that
    const int64_t min_len = std::max<int64_t>(1, (int64_t)std::ceil((double)ctx->opt.head_density * f->k));
    const int64_t split_len =
        std::max<int64_t>(1, (int64_t)std::ceil(kSplitDensity * (double)ctx->opt.head_density * f->k));
    HIPCHK(ctx, ivf_offsets(f->d, f->T, w, min_len, f->seg, f->mid, f->head, hterm, split_len, f->tlen, f->srow, sterm,
                            meta, ctx->stream));
    const bool split = X && f->srow && split_possible(ctx->opt) && X->n > 0 && X->nnz > 0;
    if (split) HIPCHK(ctx, split_sample(X->col, X->nnz, f->srow, meta, ctx->stream));
    int64_t* h = (int64_t*)ctx->pin;
    HIPCHK(ctx, hipMemcpyAsync(h, meta, kMeta * sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(ctx, hipMemcpyAsync(h + kMeta, f->seg + f->d * f->T, sizeof(int64_t), hipMemcpyDeviceToHost, ctx->stream));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    f->nmv = (int32_t)h[0];
    const int64_t P = h[1], P2 = h[kMeta], H = f->head ? h[2] : 0, SH = f->srow ? h[4] : 0;
    if (P != P2)
        return fail(ctx, SIVF_E_HIP, "internal: %lld postings for %lld centroid entries", (long long)P2, (long long)P);
    f->P = P;
    STCHK(postings_reserve(ctx, f, P));
    HIPCHK(ctx, ivf_fill(f->cur, f->k, f->d, f->kt, f->T, f->iperm, cscan, f->nmv, P, w, f->cid, f->v32, f->v16,
                         f->v64, ctx->stream));
    f->H = 0;
    f->srows = 0;
    f->sfrac = split && h[6] > 0 ? (double)h[5] / (double)h[6] : 0.0;
    const int64_t kpad = (int64_t)f->T * head_ktp(f->kt), esz = f->pdt == SIVF_BF16 ? 2 : 4;
    // room for n rows in one of the two row buffers (cap: in values); the sliced
    // rows are optional
    auto rows_reserve = [&](void** buf, int64_t* cap, int64_t n, bool optional) -> sivf_status {
        if (n * kpad <= *cap) return SIVF_OK;
        HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
        dev_free(ctx, *buf, (size_t)(*cap * esz), &f->bytes);
        *buf = nullptr;
        *cap = 0;
        const int64_t c = std::min<int64_t>(n + n / 8 + 16, std::min<int64_t>(f->d, kHeadMaxBytes / (kpad * esz))) * kpad;
        if (!optional) STCHK(dev_alloc(ctx, buf, (size_t)(c * esz), &f->bytes));
        else if (!optional_alloc(ctx, buf, (size_t)(c * esz), &f->bytes)) return SIVF_E_NOMEM;
        *cap = c;
        return SIVF_OK;
    };
    if (H > 0) {
        // every row is addressed through a descriptor of its own, so the rows
        // together may exceed 4 GiB; kHeadMaxBytes only bounds the request
        if (H * kpad * esz > kHeadMaxBytes)
            return fail(ctx, SIVF_E_UNSUPPORTED,
                        "dense head rows would take %lld bytes (%lld rows), above %lld; raise head_density",
                        (long long)(H * kpad * esz), (long long)H, (long long)kHeadMaxBytes);
        STCHK(rows_reserve(&f->hval, &f->hcap, H, false));
        HIPCHK(ctx, head_fill(hterm, f->seg, f->cid, f->v32, f->v16, f->T, head_ktp(f->kt), H, f->hval, ctx->stream));
        f->H = H;
    }
    HIPCHK(ctx, seg_records(f->seg, f->mid, f->H > 0 ? f->head : nullptr, f->d, f->T, f->rec, ctx->stream));
    // sliced rows, if a split walk pays and there is room for them
    // (the last requests of an update: they are optional)
    uint32_t* wt = nullptr;
    int32_t* sterm2 = nullptr;
    if (split && SH >= kSplitMinRows && split_pays(f->sfrac * X->nnz / X->n, X->n, f->k, f->T) && SH <= kSplitMaxRows &&
        SH * kpad * esz <= kHeadMaxBytes && SH * f->T <= kMaxGroups &&
        rows_reserve(&f->sval, &f->scap, SH, true) == SIVF_OK &&
        ws_optional(ctx, {{"split_wt", (size_t)SH * 4, (void**)&wt}, {"split_term2", (size_t)SH * 4, (void**)&sterm2}})) {
        HIPCHK(ctx, split_order(sterm, f->seg, f->T, f->v32, SH, wt, sterm2, f->srow, meta, ctx->stream));
        HIPCHK(ctx, split_fill(sterm2, f->seg, f->cid, f->v32, f->T, head_ktp(f->kt), SH, f->sval, ctx->stream));
        f->srows = SH;
    }
    // norm bounds for the signed-data certificate: needed whenever the X of a
    // later call has a negative value, whatever the centroids' signs
    if (norms) HIPCHK(ctx, centroid_norms(f->cur, f->k, f->cnorm, ctx->stream));
    f->built = true;
    return SIVF_OK;
}

// ------------------------------------------------------------ step bodies
// The ABI entry points validate their arguments (X on every call) and then
// run these; the Lloyd driver validates X once and calls them directly.

sivf_status init_impl(sivf_ctx* ctx, const Csr& Xc, int32_t k, const int32_t* init_ids_host, sivf_ivf** out) {
    if (k < 1 || k > Xc.n) return fail(ctx, SIVF_E_SHAPE, "need 1 <= k <= N (k=%d, N=%lld)", k, (long long)Xc.n);
    for (int32_t j = 0; j < k; ++j)
        if (init_ids_host[j] < 0 || init_ids_host[j] >= Xc.n)
            return fail(ctx, SIVF_E_RANGE, "init id %d at position %d outside [0, N)", init_ids_host[j], j);
    sivf_ivf* f = nullptr;
    STCHK(new_file(ctx, k, Xc.d, &f));
    f->nonneg = Xc.nonneg;
    sivf_status st = SIVF_OK;
    int32_t* ids = nullptr;
    int64_t *lens = nullptr, *scan = nullptr, *sws = nullptr;
    if (st == SIVF_OK) st = ws(ctx, "init_ids", k, &ids);
    if (st == SIVF_OK) st = ws(ctx, "init_lens", k, &lens);
    if (st == SIVF_OK) st = ws(ctx, "init_scan", k + 1, &scan);
    if (st == SIVF_OK) st = ws(ctx, "scan_ws", scan_ws_elems(k + 1) + 8, &sws);
    int64_t total = 0;
    auto H = [&](hipError_t e) {
        if (st == SIVF_OK && e != hipSuccess) st = fail(ctx, SIVF_E_HIP, "HIP error: %s", hipGetErrorString(e));
    };
    if (st == SIVF_OK) {
        H(hipMemcpyAsync(ids, init_ids_host, (size_t)k * 4, hipMemcpyHostToDevice, ctx->stream));
        H(gather_rows(Xc, ids, k, f->cur, lens, ctx->stream, 0));
        H(exclusive_scan_i64(lens, scan, k, sws, ctx->stream));
        H(hipMemcpyAsync(ctx->pin, scan + k, 8, hipMemcpyDeviceToHost, ctx->stream));
        H(hipStreamSynchronize(ctx->stream));
        total = *(const int64_t*)ctx->pin;
    }
    if (st == SIVF_OK) st = store_reserve(ctx, f, &f->cur, &f->cur_mem, total);
    if (st == SIVF_OK) {
        H(hipMemcpyAsync(f->cur.start, scan, (size_t)k * 8, hipMemcpyDeviceToDevice, ctx->stream));
        H(gather_rows(Xc, ids, k, f->cur, lens, ctx->stream, 1));
        H(fill_u8(f->lam, 0, k, ctx->stream));
    }
    if (st == SIVF_OK) st = restructure(ctx, f, true, 0.0, &Xc);
    if (st == SIVF_OK) H(hipStreamSynchronize(ctx->stream));
    if (st != SIVF_OK) {
        free_file(ctx, f);
        return st;
    }
    *out = f;
    return SIVF_OK;
}

// lambda: device flags (NULL = all moving), copied into the file
sivf_status build_impl(sivf_ctx* ctx, const sivf_csr* C, const uint8_t* lambda, sivf_ivf** out) {
    STCHK(check_csr_args(ctx, C, "centroids"));
    if (C->val_dtype != SIVF_F64) return fail(ctx, SIVF_E_INVALID, "centroid values must be SIVF_F64");
    if (C->n_rows < 1 || C->n_rows > INT32_MAX) return fail(ctx, SIVF_E_SHAPE, "need 1 <= k <= 2^31-1");
    unsigned long long* flags = nullptr;
    STCHK(ws(ctx, "vflags", 8, &flags));
    int nonneg = 1;
    STCHK(check_csr(ctx, C, "centroids", flags, &nonneg));
    const int32_t k = (int32_t)C->n_rows;
    sivf_ivf* f = nullptr;
    STCHK(new_file(ctx, k, C->n_cols, &f));
    f->nonneg = nonneg;
    sivf_status st = store_reserve(ctx, f, &f->cur, &f->cur_mem, C->nnz);
    if (st == SIVF_OK) {
        hipError_t e = csr_to_store(C->row_ptr, C->col, (const double*)C->val, k, C->nnz, f->cur, ctx->stream);
        if (e == hipSuccess)
            e = lambda ? hipMemcpyAsync(f->lam, lambda, (size_t)k, hipMemcpyDeviceToDevice, ctx->stream)
                       : fill_u8(f->lam, 0, k, ctx->stream);
        if (e != hipSuccess) st = fail(ctx, SIVF_E_HIP, "HIP error: %s", hipGetErrorString(e));
    }
    if (st == SIVF_OK) st = restructure(ctx, f, true, (double)C->nnz, nullptr);
    if (st == SIVF_OK && hipStreamSynchronize(ctx->stream) != hipSuccess) st = fail(ctx, SIVF_E_HIP, "sync failed");
    if (st != SIVF_OK) {
        free_file(ctx, f);
        return st;
    }
    *out = f;
    return SIVF_OK;
}

// The assignment step's workspace (everything it reads or writes besides
// its inputs, outputs and the file).
struct AssignBufs {
    unsigned long long* counters = nullptr;
    int32_t *a_new = nullptr, *qobj = nullptr, *qcand = nullptr, *qcnt = nullptr, *fobj = nullptr;
    float* own_new = nullptr;
    uint8_t* changed = nullptr;
    double *obj_partial = nullptr, *obj = nullptr, *obj64_partial = nullptr;
    double *st_theta = nullptr, *st_best = nullptr, *own64_cur = nullptr;
    int32_t *st_bj = nullptr, *st_cnt = nullptr, *st_cj = nullptr, *own64_queue = nullptr;
    float* st_cr = nullptr;
    uint8_t* st_rel = nullptr;
    int64_t qcap = 0;
    int nfin = 0, launches = 0, tpl = 0, nobj = 0;
    // split walk: objects per range (0: not split) and ranges
    int64_t range = 0, ranges = 1;
    uint2* ent = nullptr;
    int64_t npairs = 0;
    uint2 *hdr = nullptr, *ghdr = nullptr;
    int32_t* place = nullptr;
    float* S = nullptr;
};

// Decide whether the walk of Xc against f is split, and into which ranges.
// A range's sums take at most 4 GiB (2,000,000 objects, k = 10,000: 210 ms;
// with 1 GiB 215, with 256 MiB 270, its launches being short then).
sivf_status split_plan(sivf_ctx* ctx, Work& w, const Csr& Xc, const sivf_ivf* f, AssignBufs* b) {
    b->range = 0;
    b->ranges = 1;
    if (w.mode != Work::kCtx || !split_possible(ctx->opt) || f->srows == 0 || Xc.n == 0) return SIVF_OK;
    const double h = f->sfrac * Xc.nnz / Xc.n;
    if (!split_pays(h, Xc.n, f->k, f->T)) return SIVF_OK;
    const int64_t ktp = head_ktp(f->kt);
    int64_t pairs = 0, *most = nullptr;
    STCHK(w.get("split_most", 1, &most));
    sivf_status st = SIVF_OK;
    auto longest = [&](int64_t r, int64_t* nnz) -> sivf_status {
        *nnz = Xc.nnz;
        if (r == Xc.n) return SIVF_OK;
        HIPCHK(ctx, fill_i64(most, 0, 1, ctx->stream));
        HIPCHK(ctx, range_nnz(Xc.rp, Xc.n, r, most, ctx->stream));
        HIPCHK(ctx, hipMemcpyAsync(ctx->pin, most, 8, hipMemcpyDeviceToHost, ctx->stream));
        HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
        *nnz = *(const int64_t*)ctx->pin;
        return SIVF_OK;
    };
    const int64_t range = split_range(
        std::min<int64_t>(Xc.n, (int64_t)(1ll << 30) / ktp), [&](int64_t r) { return split_pays(h, r, f->k, f->T); },
        [&](int64_t r) {
            int64_t nnz = 0;
            st = longest(r, &nnz);
            return st == SIVF_OK ? nnz : -1;
        },
        &pairs);
    if (st != SIVF_OK || range == 0) return st;
    b->npairs = pairs;
    b->range = range;
    b->ranges = (Xc.n + range - 1) / range;
    return SIVF_OK;
}

// What a split walk needs besides assign_buffers', asked for after those.
// Without the memory the walk is not split.
void split_reserve(sivf_ctx* ctx, const sivf_ivf* f, AssignBufs* b) {
    if (!b->range) return;
    const size_t r = (size_t)b->range;
    if (ws_optional(ctx, {{"split_ent", (size_t)b->npairs * sizeof(uint2), (void**)&b->ent},
                          {"split_hdr", r * sizeof(uint2), (void**)&b->hdr},
                          {"split_ghdr", r * sizeof(uint2), (void**)&b->ghdr},
                          {"split_place", r * sizeof(int32_t), (void**)&b->place},
                          {"split_S", r * head_ktp(f->kt) * sizeof(float), (void**)&b->S}}))
        return;
    b->range = 0;
    b->ranges = 1;
}

sivf_status assign_buffers(sivf_ctx* ctx, Work& w, int64_t n, const sivf_ivf* f, AssignBufs* b) {
    const int32_t k = f->k, T = f->T;
    const int relaxed = ctx->opt.filter_mode == SIVF_MODE_RELAXED;
    b->qcap = std::max<int64_t>(1024, n / 4);
    b->nfin = (int)std::min<int64_t>(1024, std::max<int64_t>(1, (n + 4095) / 4096));
    b->tpl = std::min<int>(T, std::max<int>(1, ctx->opt.tiles_per_launch));
    b->launches = (T + b->tpl - 1) / b->tpl;
    b->nobj = ctx->n_cu * 16;   // workgroups of the exact objective (fixed: a fixed summation order)
    STCHK(w.get("counters", 16 + b->launches * b->ranges, &b->counters));
    STCHK(w.get("a_new", n, &b->a_new));
    STCHK(w.get("own_new", n, &b->own_new));
    STCHK(w.get("qobj", b->qcap, &b->qobj));
    STCHK(w.get("qcand", b->qcap * kCandCap, &b->qcand));
    STCHK(w.get("qcnt", b->qcap, &b->qcnt));
    STCHK(w.get("fobj", std::max<int64_t>(n, 1), &b->fobj));
    STCHK(w.get("changed", k, &b->changed));
    STCHK(w.get("obj_partial", b->nfin + 1, &b->obj_partial));
    b->obj = (double*)(b->counters + 12);   // read back with the counters
    if (ctx->opt.exact_objective) STCHK(w.get("obj64_partial", b->nobj, &b->obj64_partial));
    // (for all objects, also where ranges of them would do: the walk may yet turn
    // out not to be split)
    const int64_t m = std::max<int64_t>(n, 1);
    if (b->launches > 1) {
        STCHK(w.get("st_theta", m, &b->st_theta));
        STCHK(w.get("st_best", m, &b->st_best));
        STCHK(w.get("st_bj", m, &b->st_bj));
        STCHK(w.get("st_cnt", m, &b->st_cnt));
        STCHK(w.get("st_cj", m * kCandCap, &b->st_cj));
        STCHK(w.get("st_cr", m * kCandCap, &b->st_cr));
    }
    if (relaxed) {
        STCHK(w.get("own64_cur", m, &b->own64_cur));
        STCHK(w.get("own64_queue", m, &b->own64_queue));
        if (b->launches > 1) STCHK(w.get("st_rel", m, &b->st_rel));
    }
    return SIVF_OK;
}

// Validates X and, where its shape fits the file, the ids in [0, k) with it
// (nullptr: none).
sivf_status validate_with_ids(sivf_ctx* ctx, const sivf_csr* X, const sivf_ivf* f, const int32_t* ids, const char* what,
                              Csr* out, Work& w) {
    if (!ids || !X || X->n_cols != f->d) return validate(ctx, X, out, w);
    return validate(ctx, X, out, w, {{ids, X->n_rows, f->k, what}});
}

// ---------------------------------------------------------------- soft form
// Memory of a forward of Xc against k centroids by plan p; lds: with the
// commonest terms in LDS, if that pays and there is memory.
sivf_status soft_fwd_reserve(sivf_ctx* ctx, const Csr& Xc, int32_t k, const SoftFwdPlan& p, bool lds, SoftFwdWs* w,
                             double** loss) {
    const int64_t nblk = ((int64_t)k + kSoftBlk - 1) / kSoftBlk;
    *w = SoftFwdWs{};
    w->rows = p.rows;
    w->blocks = p.blocks;
    // (fewer rows per launch; without a workspace cap)
    const int64_t lds_rows =
        lds && ctx->opt.workspace_cap_bytes == 0 ? std::min(soft_lds_rows(Xc.n, Xc.nnz, Xc.d, k), w->rows) : 0;
    const int64_t least = lds_rows > 0 ? lds_rows : w->rows;
    STCHK(ws(ctx, "soft_CT", p.blocks * kSoftBlk * Xc.d, &w->CT));
    STCHK(ws(ctx, "soft_loss", 1, loss));
    STCHK(ws(ctx, "soft_pmax", w->rows * nblk, &w->pmax));
    STCHK(ws(ctx, "soft_psum", w->rows * nblk, &w->psum));
    STCHK(ws(ctx, "soft_part", Xc.n / 256 + Xc.n / least + 2, &w->part));
    const size_t d = (size_t)Xc.d;
    if (lds_rows > 0 &&
        ws_optional(ctx, {{"soft_hdr", lds_rows * sizeof(uint2), (void**)&w->hdr},
                          {"soft_count", d * 4, (void**)&w->count},
                          {"soft_slot", d * 4, (void**)&w->slot},
                          {"soft_hot", (kSplitHot + 1) * 4, (void**)&w->term},
                          {"soft_ent", (size_t)split_pairs(Xc.nnz, lds_rows) * sizeof(uint2), (void**)&w->ent}})) {
        w->nnz = Xc.nnz;
        w->nhot = w->term + kSplitHot;
        w->rows = lds_rows;
    }
    return SIVF_OK;
}

struct SoftBwd {
    SoftPlan p{};
    std::vector<int64_t> offs;   // first nonzero of each chunk of rows, and the end
    int64_t nnz_max = 0;
    float *CT = nullptr, *dS = nullptr, *dxp = nullptr, *dCT = nullptr;
    int64_t* colptr = nullptr;
    SortWs<float> sort{};
    DctWs dct{};
};

// The attempt-th plan of a backward of Xc against k centroids and its memory.
sivf_status soft_bwd_reserve(sivf_ctx* ctx, const Csr& Xc, int32_t k, int attempt, bool want_dC, bool want_dx, SoftBwd* b) {
    const int64_t n = Xc.n, d = Xc.d, nblk = ((int64_t)k + kSoftBlk - 1) / kSoftBlk;
    hipStream_t s = ctx->stream;
    SoftPlan& p = b->p;
    if (!soft_bwd_plan(attempt, n, Xc.nnz, d, nblk, &p)) return fail(ctx, SIVF_E_NOMEM, "no memory for one row");
    // nonzero offsets of the row chunks
    int64_t nch = 0;
    for (;; p.rows = (p.rows + 1) / 2) {
        nch = std::max<int64_t>(1, (n + p.rows - 1) / p.rows);
        b->offs.assign((size_t)nch + 1, 0);
        b->offs[(size_t)nch] = Xc.nnz;
        if (nch > 1) {
            int64_t* offs = nullptr;
            STCHK(ws(ctx, "soft_offs", nch + 1, &offs));
            HIPCHK(ctx, soft_chunk_offsets(Xc.rp, n, p.rows, nch, offs, s));
            HIPCHK(ctx, hipMemcpyAsync(b->offs.data(), offs, (size_t)(nch + 1) * 8, hipMemcpyDeviceToHost, s));
            HIPCHK(ctx, hipStreamSynchronize(s));
        }
        b->nnz_max = 0;
        for (size_t j = 0; j < (size_t)nch; ++j) b->nnz_max = std::max(b->nnz_max, b->offs[j + 1] - b->offs[j]);
        if (b->nnz_max <= kSoftChunkNnz || p.rows == 1) break;
    }
    p.blocks = soft_bwd_blocks(p.blocks, b->nnz_max);
    const int64_t kp = p.blocks * kSoftBlk, groups = (nblk + p.blocks - 1) / p.blocks;
    STCHK(ws(ctx, "soft_CT", kp * d, &b->CT));
    if (want_dx && nblk > 1) STCHK(ws(ctx, "soft_dxp", b->nnz_max * p.blocks, &b->dxp));
    if (!want_dC) return SIVF_OK;
    DctWs& w = b->dct;
    STCHK(ws(ctx, "soft_dS", p.rows * kp, &b->dS));
    STCHK(ws(ctx, "soft_dCT", kp * d, &b->dCT));
    STCHK(sort_ws(ctx, "soft", p.whole ? Xc.nnz : b->nnz_max, true, &b->sort));
    STCHK(ws(ctx, "csc_ptr", d + 1, &b->colptr));
    // a range of more than kSoftPiece entries has less than one piece per
    // kSoftPiece / 2 entries
    w.max_pieces = b->nnz_max / (kSoftPiece / 2);
    STCHK(ws(ctx, "dct_next", d, &w.next));
    STCHK(ws(ctx, "dct_lo", d, &w.lo));
    STCHK(ws(ctx, "dct_len", d, &w.len));
    STCHK(ws(ctx, "dct_mid", d, &w.mid));
    STCHK(ws(ctx, "dct_longt", d, &w.longt));
    STCHK(ws(ctx, "dct_longp", d, &w.longp));
    STCHK(ws(ctx, "dct_piece", w.max_pieces, &w.piece));
    STCHK(ws(ctx, "dct_piece_len", w.max_pieces, &w.piece_len));
    STCHK(ws(ctx, "dct_part", w.max_pieces * kp, &w.part));
    STCHK(ws(ctx, "dct_count", 4, &w.count));
    // the densest terms by matrix products: without a workspace cap, and only if
    // there is memory
    if (ctx->opt.workspace_cap_bytes == 0 && p.whole && n > 0 && soft_prod_may(n, Xc.nnz, k)) {
        const size_t room = (size_t)dct_cands(Xc.nnz, n);
        const int64_t last = nblk - (groups - 1) * p.blocks;   // blocks of the last group
        const size_t prod = (size_t)std::max(dct_prod_elems(p.rows, (int32_t)std::min<int64_t>(k, kp)),
                                             dct_prod_elems(p.rows, (int32_t)std::min<int64_t>(k, last * kSoftBlk)));
        w.nnz = Xc.nnz;
        ws_optional(ctx, {{"dct_prod", prod * 4, (void**)&w.prod},
                          {"dct_slot", (size_t)d * 4, (void**)&w.slot},
                          {"dct_term", kDctDense * 4, (void**)&w.term},
                          {"dct_cand", room * 4, (void**)&w.cand},
                          {"dct_cand_df", room * 4, (void**)&w.cand_df},
                          {"dct_ndense", 2 * 8, (void**)&w.ndense},
                          {"dct_xd", (size_t)p.rows * kDctDense * 4, (void**)&w.xd}});
    }
    return SIVF_OK;
}

sivf_status soft_bwd_run(sivf_ctx* ctx, const Csr& Xc, const float* C, int32_t k, float tau, const float* lse, float grad,
                         float* dC, float* dX, const SoftBwd& b) {
    const int64_t n = Xc.n, d = Xc.d, rc = b.p.rows, gk = b.p.blocks * kSoftBlk;
    hipStream_t s = ctx->stream;
    const float* xv = (const float*)Xc.val;
    const int32_t* xt_row = nullptr;
    const float* xt_val = nullptr;
    const DctWs& w = b.dct;
    // the column copy of rows [c0, c1), whose nonzeros are [p0, p1)
    auto copy = [&](int64_t c0, int64_t c1, int64_t p0, int64_t p1) -> sivf_status {
        const int32_t* xt_col = nullptr;
        SortIn<float> in{};
        in.kind = kSortCsr;
        in.n = p1 - p0;
        in.key = Xc.col + p0;
        in.val = xv + p0;
        in.rows = c1 - c0;
        in.rp = Xc.rp + c0;
        in.p0 = p0;
        in.row0 = c0;
        HIPCHK(ctx, sort_entries(in, d, b.sort, &xt_col, &xt_row, &xt_val, s));
        HIPCHK(ctx, sort_starts(xt_col, in.n, d, b.colptr, s));
        return SIVF_OK;
    };
    if (dC) {
        if (n == 0) HIPCHK(ctx, fill_i32((int32_t*)dC, 0, (int64_t)k * d, s));
        if (b.p.whole) STCHK(copy(0, n, 0, Xc.nnz));
        if (w.xd) {
            HIPCHK(ctx, fill_u64(w.ndense, 0ull, 2, s));
            HIPCHK(ctx, dct_pick(n, d, k, b.colptr, w, s));
        }
    }
    for (int64_t j0 = 0; j0 < k && n > 0; j0 += gk) {   // columns j0 .. j0 + kg - 1
        const int32_t kg = (int32_t)std::min<int64_t>(gk, k - j0);
        HIPCHK(ctx, soft_pack(C + j0 * d, b.CT, kg, d, s));
        for (int64_t c0 = 0, j = 0; c0 < n; c0 += rc, ++j) {
            const int64_t c1 = std::min(n, c0 + rc), p0 = b.offs[(size_t)j], p1 = b.offs[(size_t)j + 1];
            HIPCHK(ctx, soft_bwd_rows(c0, c1, p0, p1, Xc.rp, Xc.col, xv, b.CT, d, kg, tau, grad, lse, b.dS, b.dxp, dX,
                                      j0 > 0, ctx->n_cu, s));
            if (!dC) continue;
            HIPCHK(ctx, fill_u64(w.count, 0ull, 4, s));
            if (!b.p.whole) STCHK(copy(c0, c1, p0, p1));
            if (w.xd) HIPCHK(ctx, dct_dense_rows(c0, c1, Xc.rp, Xc.col, xv, w, ctx->n_cu, s));
            HIPCHK(ctx, soft_dct(d, kg, c0, c1, j == 0, j == 0 || !b.p.whole, b.colptr, xt_row, xt_val, b.dS, b.dCT, w,
                                 ctx->n_cu, s));
        }
        if (dC) HIPCHK(ctx, soft_unpack(b.dCT, dC + j0 * d, kg, d, s));
    }
    return SIVF_OK;
}

// The structure of a file whose update failed half way is not there to be read.
sivf_status check_built(sivf_ctx* ctx, const sivf_ivf* f) {
    if (f->built) return SIVF_OK;
    return fail(ctx, SIVF_E_INVALID, "the file has no structure since an update of it failed; update it again");
}

// Assignment step r = iter (Alg. 4) of X against the file f.
sivf_status assign_impl(sivf_ctx* ctx, Work& w, const Csr& Xc, const sivf_ivf* f, int32_t iter, int32_t* assign_inout,
                        float* own_sim_inout, double* own64_inout, uint8_t* lambda_out, sivf_iter_stats* stats_host) {
    if (Xc.d != f->d) return fail(ctx, SIVF_E_SHAPE, "X has %lld columns, centroids %lld", (long long)Xc.d, (long long)f->d);
    const int64_t n = Xc.n;
    const int32_t k = f->k;
    const int relaxed = ctx->opt.filter_mode == SIVF_MODE_RELAXED;
    const int icp_on = iter >= 2 && ctx->opt.filter_mode != SIVF_MODE_IVF;
    AssignBufs B;
    STCHK(split_plan(ctx, w, Xc, f, &B));
    STCHK(assign_buffers(ctx, w, n, f, &B));
    split_reserve(ctx, f, &B);
    const int64_t qcap = B.qcap;
    unsigned long long* counters = B.counters;
    int32_t *a_new = B.a_new, *qobj = B.qobj, *qcand = B.qcand, *qcnt = B.qcnt, *fobj = B.fobj;
    float* own_new = B.own_new;
    uint8_t* changed = B.changed;
    double *obj_partial = B.obj_partial, *obj = B.obj;
    const int nfin = B.nfin, tpl = B.tpl, launches = B.launches, nobj = B.nobj;
    double* obj64_partial = B.obj64_partial;

    WalkArgs A{};
    A.n = n;
    A.rp = Xc.rp;
    A.col = Xc.col;
    A.xval = Xc.val;
    A.x_f64 = Xc.f64;
    A.k = k;
    A.kt = f->kt;
    A.T = f->T;
    A.seg = f->seg;
    A.mid = f->mid;
    A.rec = f->rec;
    A.d = f->d;
    A.perm = f->perm;
    A.nmv = f->nmv;
    A.cid = f->cid;
    A.pval = f->pdt == SIVF_BF16 ? (const void*)f->v16 : (const void*)f->v32;
    A.lam = f->lam;
    A.cnorm = f->cnorm;
    A.a_prev = assign_inout;
    A.own_prev = own_sim_inout;
    A.icp_on = icp_on;
    A.cbicp = ctx->opt.filter_mode == SIVF_MODE_CBICP;
    A.nonneg = Xc.nonneg && f->nonneg;
    A.certify = ctx->opt.certify;
    A.eta_val = f->pdt == SIVF_BF16 ? (0x1p-8 + 0x1p-24 + 0x1p-32) : 0x1p-24;
    A.eta_x = Xc.f64 ? 0x1p-24 : 0.0;
    A.a_new = a_new;
    A.own_new = own_new;
    A.qobj = qobj;
    A.qcand = qcand;
    A.qcnt = qcnt;
    A.fobj = fobj;
    A.counters = counters;
    A.qcap = qcap;
    A.st_theta = B.st_theta;
    A.st_best = B.st_best;
    A.st_bj = B.st_bj;
    A.st_cnt = B.st_cnt;
    A.st_cj = B.st_cj;
    A.st_cr = B.st_cr;
    A.st = f->cur;
    A.relaxed = relaxed;
    A.own64_prev = own64_inout;
    A.own64_cur = B.own64_cur;
    A.st_rel = B.st_rel;
    int32_t* own64_queue = B.own64_queue;
    A.head = f->H > 0 ? f->head : nullptr;
    A.hval = f->hval;
    A.kpad = (int64_t)f->T * head_ktp(f->kt);

    hipStream_t s = ctx->stream;
    HIPCHK(ctx, fill_u64(counters, 0ull, 16 + launches * B.ranges, s));
    HIPCHK(ctx, fill_u8(changed, 0, k, s));
    HIPCHK(ctx, hipEventRecord(ctx->ev[0], s));
    if (n > 0) {
        const int bf16 = f->pdt == SIVF_BF16;
        const double terms = (double)Xc.nnz / (double)n * (B.range ? 1.0 - f->sfrac : 1.0);
        const int bpc = walk_blocks_per_cu(f->kt, bf16, A.cbicp, B.range > 0);
        if (B.range) {
            WalkArgs R = A;
            R.srow = f->srow;
            R.sval = f->sval;
            R.srows = f->srows;
            R.meta = f->meta;
            R.tlen = f->tlen;
            R.ent = B.ent;
            R.npairs = B.npairs;
            R.hdr = B.hdr;
            R.ghdr = B.ghdr;
            R.place = B.place;
            R.S = B.S;
            for (int64_t r = 0; r < B.ranges; ++r) {
                R.c0 = r * B.range;
                R.n = std::min(B.range, n - R.c0);
                HIPCHK(ctx, walk_prep(R, ctx->n_cu, s));
                for (int t = 0; t < f->T; ++t) {
                    HIPCHK(ctx, walk_dense(R, t, ctx->n_cu, s));
                    HIPCHK(ctx, walk_fast(R, terms, bf16, ctx->n_cu * bpc * kWalkWaves, t, t + 1, counters + 16 + r * f->T + t, s));
                }
            }
        } else {
            for (int l = 0; l < launches; ++l)
                HIPCHK(ctx, walk_fast(A, terms, bf16, ctx->n_cu * bpc * kWalkWaves, l * tpl, std::min(f->T, (l + 1) * tpl),
                                      counters + 16 + l, s));
        }
    }
    HIPCHK(ctx, hipEventRecord(ctx->ev[1], s));
    if (n > 0) {
        HIPCHK(ctx, rescore_candidates(A, f->cur, (int64_t)ctx->n_cu * 16, s));
        HIPCHK(ctx, rescore_full(A, f->v64, f->cur, (int64_t)ctx->n_cu * 4, s));
        if (relaxed) HIPCHK(ctx, own64_update(A, own64_inout, own64_queue, (int64_t)ctx->n_cu * 16, s));
        HIPCHK(ctx, finalize_assign(n, iter, a_new, own_new, assign_inout, own_sim_inout, changed, counters,
                                    obj_partial, nfin, s));
    }
    HIPCHK(ctx, finalize_lambda(k, iter, changed, lambda_out, counters, obj_partial, n > 0 ? nfin : 0, obj, s));
    HIPCHK(ctx, hipEventRecord(ctx->ev[2], s));
    // the FP64 objective of the new assignment against the centroids it was
    // made with, F(a^[r], mu^[r-1]) (opt-in; outside the step's timing)
    if (ctx->opt.exact_objective)
        HIPCHK(ctx, objective64(A, f->cur, assign_inout, obj64_partial, nobj, obj + 1, s));
    if (stats_host) {
        const unsigned long long* c = (const unsigned long long*)ctx->pin;
        const double* o = (const double*)(c + 12);
        HIPCHK(ctx, hipMemcpyAsync(ctx->pin, counters, 14 * sizeof(*c), hipMemcpyDeviceToHost, s));
        HIPCHK(ctx, hipStreamSynchronize(s));
        memset(stats_host, 0, sizeof(*stats_host));
        stats_host->iter = iter;
        stats_host->multadds = (int64_t)c[0];
        stats_host->rescored_objects = (int64_t)std::min<unsigned long long>(c[1], (unsigned long long)qcap);
        stats_host->full_rescored = (int64_t)c[2];
        stats_host->icp_objects = (int64_t)c[3];
        stats_host->rescored_candidates = (int64_t)c[4];
        stats_host->moved = (int64_t)c[5];
        stats_host->n_invariant = (int32_t)c[6];
        stats_host->objective_fast = o[0];
        stats_host->objective = ctx->opt.exact_objective ? o[1] : NAN;
        stats_host->head_rows = f->H;
        stats_host->relaxed_objects = (int64_t)c[7];
        stats_host->walk_bytes = (int64_t)c[10];
        stats_host->walk_wide_bytes = (int64_t)c[11];
        stats_host->walk_launches = (int32_t)(launches * B.ranges);
        float t = 0.0f;
        HIPCHK(ctx, hipEventElapsedTime(&t, ctx->ev[0], ctx->ev[1]));
        stats_host->t_walk_ms = t;
        HIPCHK(ctx, hipEventElapsedTime(&t, ctx->ev[0], ctx->ev[2]));
        stats_host->t_assign_ms = t;
    }
    return SIVF_OK;
}

// Update step (Alg. 5): centroids from assign, file restructured by lambda.
sivf_status update_impl(sivf_ctx* ctx, const Csr& Xc, const int32_t* assign, const uint8_t* lambda, sivf_ivf* f,
                        sivf_iter_stats* stats_host) {
    if (Xc.d != f->d) return fail(ctx, SIVF_E_SHAPE, "X has %lld columns, centroids %lld", (long long)Xc.d, (long long)f->d);
    const int64_t n = Xc.n;
    const int32_t k = f->k;
    hipStream_t s = ctx->stream;
    struct Updating {
        sivf_ctx* ctx;
        Updating(sivf_ctx* c, sivf_ivf* f) : ctx(c) { ctx->updating = f; }
        ~Updating() { ctx->updating = nullptr; }
    } updating(ctx, f);
    UpdateWs w{};
    w.nslots = upd_fold_groups(ctx->n_cu);
    STCHK(ws(ctx, "u_ccount", k, &w.ccount));
    STCHK(ws(ctx, "u_cstart", k + 1, &w.cstart));
    STCHK(ws(ctx, "u_memnnz", k, &w.memnnz));
    STCHK(ws(ctx, "u_ub", k, &w.ub));
    STCHK(ws(ctx, "u_ubscan", k + 1, &w.ubscan));
    STCHK(ws(ctx, "u_work", 3, &w.work));
    STCHK(ws(ctx, "u_bigslot", k, &w.bigslot));
    STCHK(ws(ctx, "u_bigc", kFoldBig, &w.bigc));
    STCHK(ws(ctx, "u_bigr", kFoldBig, &w.bigr));
    STCHK(ws(ctx, "u_splits", kFoldBig * (kFoldRanges + 1), &w.splits));
    STCHK(ws(ctx, "u_jobs", kFoldBig * kFoldRanges, &w.jobs));
    STCHK(ws(ctx, "u_scan", scan_ws_elems(k) + 8, &w.scan_ws));
    SortWs<float> sw{};
    STCHK(sort_ws(ctx, "u_sort", n, false, &sw));
    // the accumulators and their marks start zeroed; the kernel leaves them so
    STCHK(ws_zeroed(ctx, "u_W", (int64_t)(w.nslots + kFoldBig) * Xc.d, &w.W));
    STCHK(ws_zeroed(ctx, "u_touched", (int64_t)(w.nslots + kFoldBig) * ((Xc.d + 63) / 64), &w.touched));
    HIPCHK(ctx, hipEventRecord(ctx->ev[3], s));
    HIPCHK(ctx, upd_sort(assign, n, k, Xc.rp, sw, &w, s));
    HIPCHK(ctx, upd_bounds(k, n, Xc.d, Xc.nnz, lambda, 1, f->cur, w, s));
    // room for the new entries: the exact bound is on the device; where the
    // largest it can be already fits or is small, the host need not wait for it
    // (after a failed update f->P may not be the current entries)
    int64_t most = f->P + Xc.nnz;
    if (f->d < most / k) most = f->d * k;
    if (!f->nxt.term || f->nxt.cap < most || !f->built) {
        if (ctx->opt.workspace_cap_bytes != 0 || !f->built || most > ((int64_t)4 << 20)) {
            int64_t* total = (int64_t*)ctx->pin;
            HIPCHK(ctx, hipMemcpyAsync(total, w.ubscan + k, 8, hipMemcpyDeviceToHost, s));
            HIPCHK(ctx, hipStreamSynchronize(s));
            most = *total;
        }
        STCHK(store_reserve(ctx, f, &f->nxt, &f->nxt_mem, most));
    }
    f->built = false;
    HIPCHK(ctx, upd_means(Xc, k, lambda, 1, f->cur, f->nxt, w, f->cnorm, s));
    std::swap(f->cur, f->nxt);
    std::swap(f->cur_mem, f->nxt_mem);
    HIPCHK(ctx, hipMemcpyAsync(f->lam, lambda, (size_t)k, hipMemcpyDeviceToDevice, s));
    f->nonneg = f->nonneg && Xc.nonneg;
    // (a cluster's members share terms: a quarter to two thirds of their nonzeros remain)
    STCHK(restructure(ctx, f, false, Xc.nnz / 3.0, &Xc));
    HIPCHK(ctx, hipEventRecord(ctx->ev[4], s));
    if (stats_host) {
        HIPCHK(ctx, hipStreamSynchronize(s));
        float t = 0.0f;
        HIPCHK(ctx, hipEventElapsedTime(&t, ctx->ev[3], ctx->ev[4]));
        stats_host->t_update_ms = t;
    }
    return SIVF_OK;
}

}  // namespace

// =========================================================================== ABI
extern "C" {

sivf_status sivf_default_options(sivf_options* opt) {
    if (!opt) return SIVF_E_INVALID;
    opt->posting_dtype = SIVF_F32;
    opt->filter_mode = SIVF_MODE_SIVF;
    opt->k_tile = 0;
    opt->certify = 1;
    opt->workspace_cap_bytes = 0;
    opt->head_density = -1.0f;
    opt->tiles_per_launch = 0;
    opt->exact_objective = 0;
    return SIVF_OK;
}

sivf_status sivf_create(sivf_ctx** out, int device, void* hip_stream, const sivf_options* opt) {
    if (!out) return SIVF_E_INVALID;
    *out = nullptr;
    sivf_options o;
    sivf_default_options(&o);
    if (opt) o = *opt;
    if (o.posting_dtype != SIVF_F32 && o.posting_dtype != SIVF_BF16) return SIVF_E_INVALID;
    if (o.filter_mode < 0 || o.filter_mode > 3) return SIVF_E_INVALID;
    if (o.k_tile != 0 && (o.k_tile < 64 || o.k_tile > kMaxTile || o.k_tile % 64 != 0)) return SIVF_E_INVALID;
    if (!(o.head_density <= 1.0f)) return SIVF_E_INVALID;   // NaN fails too
    // negative: the precision's own density (dense rows cost half the bytes
    // in BF16, so more terms pay for one there)
    if (o.head_density < 0.0f) o.head_density = o.posting_dtype == SIVF_BF16 ? 0.3f : 0.5f;
    if (o.tiles_per_launch < 0) return SIVF_E_INVALID;
    if (o.exact_objective != 0 && o.exact_objective != 1) return SIVF_E_INVALID;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return SIVF_E_HIP;
    sivf_ctx* ctx = new (std::nothrow) sivf_ctx();
    if (!ctx) return SIVF_E_NOMEM;
    ctx->device = device;
    ctx->stream = (hipStream_t)hip_stream;
    ctx->opt = o;
    DevGuard g(device);
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && ncu > 0)
        ctx->n_cu = ncu;
    if (scratch_setup(device) != hipSuccess) {
        (void)hipGetLastError();
        delete ctx;
        return SIVF_E_HIP;
    }
    bool ok = hipHostMalloc(&ctx->pin, kPinBytes, hipHostMallocDefault) == hipSuccess;
    for (auto& e : ctx->ev) ok = ok && hipEventCreate(&e) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        (void)sivf_destroy(ctx);
        return SIVF_E_HIP;
    }
    *out = ctx;
    return SIVF_OK;
}

sivf_status sivf_destroy(sivf_ctx* ctx) {
    if (!ctx) return SIVF_OK;
    DevGuard g(ctx->device);
    (void)hipStreamSynchronize(ctx->stream);
    for (auto& kv : ctx->ws) (void)hipFree(kv.second.p);
    for (auto& e : ctx->ev)
        if (e) (void)hipEventDestroy(e);
    if (ctx->pin) (void)hipHostFree(ctx->pin);
    delete ctx;
    return SIVF_OK;
}

const char* sivf_last_error(const sivf_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

sivf_status sivf_validate_csr(sivf_ctx* ctx, const sivf_csr* X) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    Csr c;
    return validate(ctx, X, &c);
}

sivf_status sivf_init_centroids(sivf_ctx* ctx, const sivf_csr* X, int32_t k, const int32_t* init_ids_host,
                                sivf_ivf** out) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!out || !init_ids_host) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    Csr Xc;
    STCHK(validate(ctx, X, &Xc));
    return init_impl(ctx, Xc, k, init_ids_host, out);
}

sivf_status sivf_build_centroid_ivf(sivf_ctx* ctx, const sivf_csr* C, const uint8_t* lambda, sivf_ivf** out) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!out) return fail(ctx, SIVF_E_INVALID, "NULL out");
    return build_impl(ctx, C, lambda, out);
}

sivf_status sivf_ivf_free(sivf_ctx* ctx, sivf_ivf* ivf) {
    if (!ivf) return SIVF_OK;
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    free_file(ctx, ivf);
    return SIVF_OK;
}

sivf_status sivf_ivf_sizes(sivf_ctx* ctx, const sivf_ivf* f, int32_t* k_host, int64_t* d_host, int64_t* nnz_host,
                           int32_t* n_tiles_host, int32_t* k_tile_host) {
    if (!ctx || !f) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    if (k_host) *k_host = f->k;
    if (d_host) *d_host = f->d;
    if (nnz_host) *nnz_host = f->P;
    if (n_tiles_host) *n_tiles_host = f->T;
    if (k_tile_host) *k_tile_host = f->kt;
    return SIVF_OK;
}

sivf_status sivf_ivf_export(sivf_ctx* ctx, const sivf_ivf* f, int64_t* c_ptr, int32_t* c_col, double* c_val,
                            uint8_t* lambda, int64_t* term_ptr, int32_t* split, int32_t* p_cid, double* p_val) {
    if (!ctx || !f) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if ((c_col || c_val) && !c_ptr) return fail(ctx, SIVF_E_INVALID, "c_col/c_val need c_ptr");
    if ((p_cid || p_val) && !term_ptr) return fail(ctx, SIVF_E_INVALID, "p_cid/p_val need term_ptr");
    if (term_ptr || split) STCHK(check_built(ctx, f));
    int64_t* sws = nullptr;
    STCHK(ws(ctx, "scan_ws", scan_ws_elems(std::max<int64_t>(f->k, f->d) + 1) + 8, &sws));
    if (c_ptr) {
        HIPCHK(ctx, exclusive_scan_i64(f->cur.nnz, c_ptr, f->k, sws, ctx->stream));
        if (c_col || c_val) HIPCHK(ctx, store_export(f->cur, f->k, c_ptr, c_col, c_val, ctx->stream));
    }
    if (lambda) HIPCHK(ctx, hipMemcpyAsync(lambda, f->lam, (size_t)f->k, hipMemcpyDeviceToDevice, ctx->stream));
    if (term_ptr || split) {
        int64_t* cnt = nullptr;
        STCHK(ws(ctx, "exp_cnt", f->d, &cnt));
        HIPCHK(ctx, ivf_export(f, term_ptr, split, p_cid, p_val, cnt, sws, ctx->stream));
    }
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    return SIVF_OK;
}

sivf_status sivf_assign(sivf_ctx* ctx, const sivf_csr* X, const sivf_ivf* f, int32_t iter, int32_t* assign_inout,
                        float* own_sim_inout, double* own64_inout, uint8_t* lambda_out, sivf_iter_stats* stats_host) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!f || !assign_inout || !own_sim_inout || !lambda_out) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    if (ctx->opt.filter_mode == SIVF_MODE_RELAXED && !own64_inout)
        return fail(ctx, SIVF_E_INVALID, "the RELAXED filter needs own64_inout");
    if (iter < 1) return fail(ctx, SIVF_E_INVALID, "iter must be >= 1");
    STCHK(check_built(ctx, f));
    Csr Xc;
    Work w{ctx};
    STCHK(validate_with_ids(ctx, X, f, iter >= 2 ? assign_inout : nullptr, "assign_inout (a^[r-1])", &Xc, w));
    return assign_impl(ctx, w, Xc, f, iter, assign_inout, own_sim_inout, own64_inout, lambda_out, stats_host);
}

sivf_status sivf_assign_noalloc(sivf_ctx* ctx, const sivf_csr* X, const sivf_ivf* f, int32_t iter,
                                int32_t* assign_inout, float* own_sim_inout, double* own64_inout,
                                uint8_t* lambda_out, sivf_iter_stats* stats_host) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!f || !assign_inout || !own_sim_inout || !lambda_out) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    if (ctx->opt.filter_mode == SIVF_MODE_RELAXED && !own64_inout)
        return fail(ctx, SIVF_E_INVALID, "the RELAXED filter needs own64_inout");
    if (iter < 1) return fail(ctx, SIVF_E_INVALID, "iter must be >= 1");
    STCHK(check_built(ctx, f));
    STCHK(check_csr_args(ctx, X, "X"));
    // the same requests as the run below, counted without memory
    Work m{ctx, Work::kMeasure};
    unsigned long long* flags = nullptr;
    STCHK(m.get("vflags", 8, &flags));
    AssignBufs B;
    STCHK(assign_buffers(ctx, m, X->n_rows, f, &B));
    if (m.used > kScratchBytes)
        return fail(ctx, SIVF_E_UNSUPPORTED,
                    "sivf_assign_noalloc: %lld objects against %d centroids (%d launches) need %zu bytes of "
                    "scratch, above its %zu; use sivf_assign", (long long)X->n_rows, f->k, B.launches, m.used,
                    kScratchBytes);
    void* base = scratch_of(ctx->device);
    if (!base) return fail(ctx, SIVF_E_HIP, "no scratch address for device %d", ctx->device);
    Work w{ctx, Work::kFixed, (char*)base, kScratchBytes};
    Csr Xc;
    STCHK(validate_with_ids(ctx, X, f, iter >= 2 ? assign_inout : nullptr, "assign_inout (a^[r-1])", &Xc, w));
    return assign_impl(ctx, w, Xc, f, iter, assign_inout, own_sim_inout, own64_inout, lambda_out, stats_host);
}

sivf_status sivf_update(sivf_ctx* ctx, const sivf_csr* X, const int32_t* assign, const uint8_t* lambda,
                        sivf_ivf* f, sivf_iter_stats* stats_host) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!f || !assign || !lambda) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    Csr Xc;
    Work w{ctx};
    STCHK(validate_with_ids(ctx, X, f, assign, "assign", &Xc, w));
    return update_impl(ctx, Xc, assign, lambda, f, stats_host);
}

sivf_status sivf_run_lloyd(sivf_ctx* ctx, const sivf_csr* X, int32_t k, const int32_t* init_ids_host, int32_t max_iter,
                           int32_t* assign_out, float* own_sim_out, sivf_ivf** centroids_out,
                           sivf_iter_stats* per_iter_host, int32_t* iters_done_host) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (max_iter < 1) return fail(ctx, SIVF_E_INVALID, "max_iter must be >= 1");
    if (!init_ids_host) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    // X is validated once: the driver holds the stream for the whole run
    Csr Xc;
    STCHK(validate(ctx, X, &Xc));
    sivf_ivf* f = nullptr;
    STCHK(init_impl(ctx, Xc, k, init_ids_host, &f));
    int32_t* a = assign_out;
    float* own = own_sim_out;
    uint8_t* lam = nullptr;
    sivf_status st = SIVF_OK;
    if (!a) st = ws(ctx, "lloyd_a", Xc.n, &a);
    if (st == SIVF_OK && !own) st = ws(ctx, "lloyd_own", Xc.n, &own);
    if (st == SIVF_OK) st = ws(ctx, "lloyd_lam", k, &lam);
    double* own64 = nullptr;   // exact own similarities (relaxed ICP state)
    if (st == SIVF_OK && ctx->opt.filter_mode == SIVF_MODE_RELAXED)
        st = ws(ctx, "lloyd_own64", std::max<int64_t>(Xc.n, 1), &own64);
    int32_t done = 0;
    for (int32_t r = 1; st == SIVF_OK && r <= max_iter; ++r) {
        sivf_iter_stats stt{};
        Work w{ctx};
        st = assign_impl(ctx, w, Xc, f, r, a, own, own64, lam, &stt);
        if (st != SIVF_OK) break;
        done = r;
        if (per_iter_host) per_iter_host[r - 1] = stt;
        if (r >= 2 && stt.moved == 0) break;
        if (r == max_iter) break;  // the last assignment's centroids stay as they are
        st = update_impl(ctx, Xc, a, lam, f, &stt);
        if (st != SIVF_OK) break;
        if (per_iter_host) per_iter_host[r - 1].t_update_ms = stt.t_update_ms;
    }
    if (st == SIVF_OK && hipStreamSynchronize(ctx->stream) != hipSuccess) st = fail(ctx, SIVF_E_HIP, "sync failed");
    if (iters_done_host) *iters_done_host = done;
    if (st != SIVF_OK || !centroids_out) {
        free_file(ctx, f);
        if (centroids_out) *centroids_out = nullptr;
        return st;
    }
    *centroids_out = f;
    return SIVF_OK;
}

sivf_status sivf_resume(sivf_ctx* ctx, const sivf_csr* X, const sivf_csr* centroids, const int32_t* a_prev,
                        const int32_t* a_prev2, sivf_ivf** out, float* own_sim_out, double* own64_out) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!out || !a_prev || !own_sim_out || !centroids) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    if (ctx->opt.filter_mode == SIVF_MODE_RELAXED && !own64_out)
        return fail(ctx, SIVF_E_INVALID, "the RELAXED filter needs own64_out");
    Csr Xc;
    const int32_t k = (int32_t)std::min<int64_t>(centroids->n_rows, INT32_MAX);
    if (X && X->n_cols == centroids->n_cols && k >= 1 && k <= X->n_rows) {
        if (a_prev2)
            STCHK(validate(ctx, X, &Xc, {{a_prev, X->n_rows, k, "a_prev"}, {a_prev2, X->n_rows, k, "a_prev2"}}));
        else
            STCHK(validate(ctx, X, &Xc, {{a_prev, X->n_rows, k, "a_prev"}}));
    } else {
        STCHK(validate(ctx, X, &Xc));
    }
    if (centroids->n_cols != Xc.d)
        return fail(ctx, SIVF_E_SHAPE, "X has %lld columns, centroids %lld", (long long)Xc.d,
                    (long long)centroids->n_cols);
    if (centroids->n_rows < 1 || centroids->n_rows > Xc.n)
        return fail(ctx, SIVF_E_SHAPE, "need 1 <= k <= N (k=%lld, N=%lld)", (long long)centroids->n_rows,
                    (long long)Xc.n);
    // lambda of the restart point: membership of every cluster unchanged
    // between the last two assignments (all 0 when only one exists)
    uint8_t *changed = nullptr, *lam = nullptr;
    unsigned long long* cnt = nullptr;
    double* dummy = nullptr;
    STCHK(ws(ctx, "resume_changed", k, &changed));
    STCHK(ws(ctx, "resume_lam", k, &lam));
    STCHK(ws(ctx, "resume_cnt", 16, &cnt));
    STCHK(ws(ctx, "resume_obj", 1, &dummy));
    hipStream_t s = ctx->stream;
    HIPCHK(ctx, fill_u8(changed, 0, k, s));
    HIPCHK(ctx, fill_u64(cnt, 0ull, 16, s));
    if (a_prev2 && Xc.n > 0) HIPCHK(ctx, mark_changed(Xc.n, a_prev2, a_prev, changed, s));
    HIPCHK(ctx, finalize_lambda(k, a_prev2 ? 2 : 1, changed, lam, cnt, nullptr, 0, dummy, s));
    sivf_ivf* f = nullptr;
    STCHK(build_impl(ctx, centroids, lam, &f));
    WalkArgs A{};
    A.n = Xc.n;
    A.rp = Xc.rp;
    A.col = Xc.col;
    A.xval = Xc.val;
    A.x_f64 = Xc.f64;
    if (Xc.n > 0) {
        hipError_t e = resume_own(A, f->cur, a_prev, f->lam, own_sim_out, own64_out, (int64_t)ctx->n_cu * 32, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            free_file(ctx, f);
            return fail(ctx, SIVF_E_HIP, "HIP error: %s", hipGetErrorString(e));
        }
    }
    *out = f;
    return SIVF_OK;
}

sivf_status sivf_soft_assign_fwd(sivf_ctx* ctx, const sivf_csr* X, const float* C, int32_t k, float tau, float* lse_out,
                                 double* loss_host) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!C || !lse_out) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    if (k < 1) return fail(ctx, SIVF_E_SHAPE, "k must be >= 1");
    if (!(tau > 0.0f) || !std::isfinite(tau)) return fail(ctx, SIVF_E_INVALID, "tau must be positive and finite");
    Csr Xc;
    STCHK(validate(ctx, X, &Xc));
    if (Xc.f64) return fail(ctx, SIVF_E_UNSUPPORTED, "soft assignment takes SIVF_F32 object values");
    const std::string err = ctx->err;
    double* loss = nullptr;
    SoftFwdWs w{};
    sivf_status st = SIVF_E_NOMEM;
    SoftFwdPlan p;
    for (int a = 0; st == SIVF_E_NOMEM && soft_fwd_plan(a, Xc.n, ((int64_t)k + kSoftBlk - 1) / kSoftBlk, &p); ++a) {
        if (a > 0) ws_drop(ctx, {"soft_"});
        st = soft_fwd_reserve(ctx, Xc, k, p, a == 0, &w, &loss);
    }
    if (st == SIVF_E_NOMEM) ws_drop(ctx, {"soft_"});
    STCHK(st);
    ctx->err = err;
    hipStream_t s = ctx->stream;
    HIPCHK(ctx, soft_forward(Xc.n, Xc.nnz, Xc.rp, Xc.col, (const float*)Xc.val, C, Xc.d, k, tau, lse_out, loss, w, ctx->n_cu, s));
    if (loss_host) {
        HIPCHK(ctx, hipMemcpyAsync(ctx->pin, loss, sizeof(double), hipMemcpyDeviceToHost, s));
        HIPCHK(ctx, hipStreamSynchronize(s));
        *loss_host = *(const double*)ctx->pin;
    }
    return SIVF_OK;
}

sivf_status sivf_soft_assign_bwd(sivf_ctx* ctx, const sivf_csr* X, const float* C, int32_t k, float tau, const float* lse,
                                 float grad_loss, float* dC_out, float* dxval_out) {
    if (!ctx) return SIVF_E_INVALID;
    DevGuard g(ctx->device);
    if (!C || !lse) return fail(ctx, SIVF_E_INVALID, "NULL argument");
    if (k < 1) return fail(ctx, SIVF_E_SHAPE, "k must be >= 1");
    if (!(tau > 0.0f) || !std::isfinite(tau)) return fail(ctx, SIVF_E_INVALID, "tau must be positive and finite");
    if (!std::isfinite(grad_loss)) return fail(ctx, SIVF_E_NONFINITE, "grad_loss must be finite");
    Csr Xc;
    STCHK(validate(ctx, X, &Xc));
    if (Xc.f64) return fail(ctx, SIVF_E_UNSUPPORTED, "soft assignment takes SIVF_F32 object values");
    if (!dC_out && !dxval_out) return SIVF_OK;
    const std::string err = ctx->err;
    for (int attempt = 0;; ++attempt) {
        SoftBwd b;
        const sivf_status st = soft_bwd_reserve(ctx, Xc, k, attempt, dC_out != nullptr, dxval_out != nullptr, &b);
        if (st == SIVF_OK) {
            ctx->err = err;
            return soft_bwd_run(ctx, Xc, C, k, tau, lse, grad_loss, dC_out, dxval_out, b);
        }
        if (st != SIVF_E_NOMEM) return st;
        ws_drop(ctx, {"soft_", "csc_", "dct_"});   // for the next plan, or for other calls
        SoftPlan next;
        if (!soft_bwd_plan(attempt + 1, Xc.n, Xc.nnz, Xc.d, ((int64_t)k + kSoftBlk - 1) / kSoftBlk, &next)) return st;
    }
}

}  // extern "C"
