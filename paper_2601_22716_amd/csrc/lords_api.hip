// C ABI of the library (include/lords.h): argument checks, path choice, launches.
// No arithmetic of the method lives here.
#include "../../include/lords.h"
#include "lords_launch.h"

#include <algorithm>
#include <mutex>

namespace lords {
bool fused_rank_supported(int r, bool f32fact);
}

namespace {

constexpr int kVersion = 200;   // 0.2.0
constexpr int kMaxDevices = 16;

// Layout of a workspace, the library's own or a caller's:
//   [0, kZeroBytes)                         exchange slots of the one-/two-token kernel   } zero when handed over,
//   [kZeroBytes, kZeroBytes + kTicketBytes) arrival tickets of the few-token kernels      } left at zero by every call
//   [kFront, ...)                           fp32 partial sums and other scratch, contents of no interest between calls
constexpr size_t kFront = lords::kZeroBytes + lords::kTicketBytes;

struct WsView {
    unsigned char *base = nullptr;     // start of the zero region
    size_t bytes = 0;
    void *zeroed() const { return base; }
    void *tickets() const { return base ? base + lords::kZeroBytes : nullptr; }    // what the few-token kernels call "workspace"
    void *scratch() const { return base ? base + kFront : nullptr; }
    unsigned char *f32_parts = nullptr;     // kF32Parts bytes, or null (a workspace that is not the library's own)
    // How a large product uses it: as the large-M kernel plans with what is there; by whole tiles; in two passes.
    enum Large { kShared, kWhole, kTwoPass } large = kShared;
};

// Partial sums of a large-M product with fp32 factors, the most its plan ever asks for (256 workgroups x 128 x 256 tiles).
// They have a place of their own beside the library's first block: such a call then needs the front alone, as it always
// did, also under capture, and cuts its sums the same way whatever was allocated before it.
constexpr size_t kF32Parts = (size_t)32 << 20;

// The library's own per-device workspace (convenience entry points).  A block that has been handed
// out is never freed or moved: work already queued, and HIP graphs captured earlier, keep using it.
// When a call needs more, a new block is allocated (and its front zeroed, which waits for the
// device); while the stream is being captured that is refused instead.  A refusal leaves no error
// behind: the caller may go on with less, and the launches that follow report the thread's last error.
// Where the caller can do with less (`optional`), what the device had no room for is not asked for again at once: two
// allocations that fail cost more than what they are wanted for gains, on every call beside an allocator that has taken the card.
// kAskAgain such calls later it is, as memory may have been given back.
struct OwnWorkspace {
    unsigned char *ptr = nullptr;
    size_t bytes = 0;
    unsigned char *f32_parts = nullptr;
    size_t refused = ~(size_t)0;        // the least that the device had no room for
    int without = 0;                    // calls that have done without since
};
constexpr int kAskAgain = 1000;
OwnWorkspace g_ws[kMaxDevices];
std::mutex g_ws_mutex;

int get_workspace(size_t need, void *stream, WsView *out, bool optional = false)
{
    *out = WsView{};
    if (need < kFront) need = kFront;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LORDS_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_ws_mutex);
    OwnWorkspace &w = g_ws[dev];
    if (w.bytes < need) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing((hipStream_t)stream, &cap) != hipSuccess) {
            (void)hipGetLastError();
            return LORDS_ERR_LAUNCH;
        }
        if (cap != hipStreamCaptureStatusNone) return LORDS_ERR_LAUNCH;
        const size_t behind = w.f32_parts ? 0 : kF32Parts;
        if (optional && need + behind >= w.refused) {
            if (w.without++ < kAskAgain) return LORDS_ERR_LAUNCH;
            w.refused = ~(size_t)0;
        }
        size_t want = need < (size_t)(16u << 20) ? (size_t)(16u << 20) : need + need / 2;
        unsigned char *fresh = nullptr;
        want = (want + 255) & ~(size_t)255;
        if (hipMalloc((void **)&fresh, want + behind) != hipSuccess) {
            want = (need + 255) & ~(size_t)255;            // (no room for more than was asked for)
            if (hipMalloc((void **)&fresh, want + behind) != hipSuccess) {
                (void)hipGetLastError();
                w.refused = std::min(w.refused, need + behind);
                w.without = 0;
                return LORDS_ERR_LAUNCH;
            }
            (void)hipGetLastError();
        }
        if (hipMemset(fresh, 0, kFront) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
            (void)hipFree(fresh);
            return LORDS_ERR_LAUNCH;
        }
        w.ptr = fresh;          // (the previous block stays allocated: it may still be in use)
        w.bytes = want;
        if (behind) w.f32_parts = fresh + want;
    }
    out->base = w.ptr;
    out->bytes = w.bytes;
    out->f32_parts = w.f32_parts;
    return LORDS_OK;
}

// One token: the regrouped kernel of lords_gemv.hip wherever it takes the shape.  Two tokens: the same,
// except at ranks above 32 on layers above 32 M weights with at least as many rows as columns, where the
// few-token kernel measured faster (us, regrouped / few-token: 14336 x 4096 rank 48 20.9 / 19.6,
// 28672 x 8192 rank 64 85 / 66; against 14336 x 4096 rank 32 14.7 / 15.4, 4096 x 14336 rank 32 16.7 / 17.8,
// rank 48 22.3 / 24.6, 4096 x 4096 8.3 / 10.2, 6144 x 4096 10.1 / 11.1).
bool use_gemv(const lords::MatmulProblem &p, lords_path path)
{
    if (path == LORDS_PATH_SMALLM) return false;
    if (path == LORDS_PATH_GEMV) return lords::decode_gemv_supported(p);
    if (p.M == 2 && p.r > 32 && (long)p.N * p.K > (32L << 20) && p.N >= p.K) return false;
    return lords::decode_gemv_supported(p);
}

// Which few-token kernel takes a problem, and the scratch it asks for behind the tickets.
enum DecodeKind { kFew, kFast, kGeneral };
DecodeKind decode_kind(const lords::MatmulProblem &p)
{
    if (p.M > 1 && lords::decode_mx_supported(p)) return kFew;
    if (lords::decode_fast_supported(p)) return kFast;
    return kGeneral;
}
size_t decode_scratch(const lords::MatmulProblem &p)
{
    size_t with_tickets;
    switch (decode_kind(p)) {
        case kFew: with_tickets = lords::decode_mx_workspace_bytes(p); break;
        case kFast: with_tickets = lords::decode_fast_workspace_bytes(p); break;
        default: return lords::decode_workspace_bytes(p);
    }
    return with_tickets > lords::kTicketBytes ? with_tickets - lords::kTicketBytes : 0;
}
inline bool is_decode(lords_path path) { return path == LORDS_PATH_DECODE || path == LORDS_PATH_GEMV || path == LORDS_PATH_SMALLM; }
// Measured cross-over.  Up to 16 tokens the few-token kernels win (28672 x 8192, rank 64: 68 / 80 us at
// 8 / 16 tokens against 87-90 us for the large-M kernel; 4096 x 14336, rank 48: 25 / 31 us against 50 us),
// except at ranks 65..128, which the few-token family serves with its oldest kernel: there the large-M
// kernel wins from two tokens on (28672 x 8192, rank 128: 219 against 117 us at two tokens, 235 against
// 117 us at eight; 14336 x 4096: 71 against 48 us at two; one token: 124 against 117 us and 42 against 48 us).
inline lords_path resolve_path(lords_path path, const lords::MatmulProblem &p)
{
    if (path != LORDS_PATH_AUTO) return path;
    if (p.M > 16) return LORDS_PATH_PREFILL;
    if (p.M >= 2 && p.r > 64 && lords::prefill_fast_supported(p)) return LORDS_PATH_PREFILL;
    // fp32 factors (contraction 3 r, the same oldest few-token kernel): above 32 columns on layers above 32 M weights
    // (4 bits, us, few-token / large-M at 2, 4, 16 tokens; of ten layers from 0.1 M to 235 M weights at ranks 11 to 42 the
    // large-M kernel wins on all above the line, and below it only at 16 tokens, from 16 M weights on):
    //   4096 x 4096   rank 16 24.4 / 28.1, 24.3 / 28.1, 32.1 / 28.0   rank 40 34.8 / 36.0, 34.8 / 36.2, 42.0 / 35.9
    //   8192 x 4096   rank 16 29.9 / 36.4, 32.2 / 36.7, 45.3 / 36.3   rank 40 42.7 / 44.5, 45.1 / 44.1, 57.8 / 44.3   (= 32 M)
    //   9216 x 4096   rank 16 41.2 / 38.2, 44.0 / 38.5, 59.4 / 38.6   rank 40 60.4 / 52.2, 63.3 / 52.2, 78.3 / 52.3
    //   28672 x 8192  rank 16  185 / 94,    189 / 93,    226 / 93     rank 40  279 / 184,   283 / 184,   319 / 184
    //   9216 x 4096   rank 8  28.3 / 29.9, 30.1 / 30.1, 36.1 / 30.1
    if (p.M >= 2 && p.f32fact && 3 * p.r > 32 && (long)p.N * p.K > (32L << 20) && lords::prefill_fast_supported(p)) return LORDS_PATH_PREFILL;
    // ... and beyond 128 columns at any token count, where the few-token family is left with its general kernel
    // (us, general / this: rank 43, one token, 14336 x 4096 473 / 68, 875 x 6496 73 / 43; 40 tokens 1025 / 68, 1676 / 44;
    //  rank 64, 17 tokens, 256 x 256 75 / 23).
    if (p.f32fact && 3 * p.r > 128 && lords::prefill_fast_supported(p)) return LORDS_PATH_PREFILL;
    return LORDS_PATH_DECODE;
}

// Bytes of workspace (front included) one checked problem needs on `path` (already resolved).  The
// large-M kernel takes what it is given: with `limit` bytes or more it shares tiles between
// workgroups, with less it falls back to whole tiles and needs none.
constexpr size_t kNoLimit = ~(size_t)0;
size_t matmul_need(const lords::MatmulProblem &p, lords_path path, size_t limit = kNoLimit)
{
    size_t scratch = 0;
    if (is_decode(path)) scratch = use_gemv(p, path) ? 0 : decode_scratch(p);
    else if (lords::prefill_fast_supported(p)) scratch = lords::prefill_fast_workspace_bytes(p, limit > kFront ? limit - kFront : 0);
    return kFront + ((scratch + 255) & ~(size_t)255);
}

// The least of a workspace that is to be accepted for it.
size_t matmul_least(const lords::MatmulProblem &p, lords_path path)
{
    if (is_decode(path) || !lords::prefill_fast_supported(p)) return matmul_need(p, path);
    return kFront + ((lords::prefill_least_workspace_bytes(p) + 255) & ~(size_t)255);
}

lords::BatchedProblem batch_of(const lords::MatmulProblem &p)
{
    lords::BatchedProblem bp;
    bp.X = p.X; bp.codebook = p.codebook; bp.codes[0] = p.codes; bp.B[0] = p.B; bp.A[0] = p.A; bp.Y[0] = p.Y; bp.N[0] = p.N;
    bp.L = 1; bp.M = p.M; bp.K = p.K; bp.r = p.r; bp.bits = p.bits;
    bp.f32fact = p.f32fact; bp.f32out = p.f32out; bp.act = false; bp.tiled = p.tiled;
    return bp;
}

// The matrices of a batched call for which pick(l) holds.
template <class Pick>
lords::BatchedProblem batch_where(const lords::BatchedProblem &bp, Pick pick)
{
    lords::BatchedProblem out = bp;
    out.L = 0;
    for (int l = 0; l < bp.L; ++l) {
        if (!pick(l)) continue;
        out.codes[out.L] = bp.codes[l]; out.B[out.L] = bp.B[l]; out.A[out.L] = bp.A[l]; out.Y[out.L] = bp.Y[l]; out.N[out.L] = bp.N[l];
        out.whole[out.L] = bp.whole[l];
        ++out.L;
    }
    return out;
}

// The library's own workspace for a product in two passes, and `extra` bytes behind its scratch.  Where the memory is not to
// be had (a stream that is being captured, mostly), whole tiles of the large-M kernel give the same result bit for bit.
int two_pass_workspace(const lords::BatchedProblem &bp, size_t extra, void *stream, WsView *ws, size_t *own)
{
    *own = kFront + ((lords::two_pass_workspace_bytes(bp) + 255) & ~(size_t)255);
    int rc = get_workspace(*own + extra, stream, ws, true);
    ws->large = WsView::kTwoPass;
    if (rc != LORDS_OK) {
        *own = kFront;
        rc = get_workspace(*own + extra, stream, ws);
        ws->large = WsView::kWhole;
    }
    return rc;
}

// The large-M kernel, with the scratch its problem has in this workspace, or both passes.
int launch_large(const lords::MatmulProblem &p, const WsView &ws, void *stream, const float *gate = nullptr)
{
    if (ws.large == WsView::kTwoPass && !gate)
        return lords::launch_two_pass(batch_of(p), ws.scratch(), (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
    if (ws.large != WsView::kShared)
        return lords::launch_prefill_fast(p, nullptr, 0, ws.zeroed(), (hipStream_t)stream, gate) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
    void *part = ws.scratch();
    size_t bytes = ws.bytes > kFront ? ws.bytes - kFront : 0;
    if (p.f32fact && ws.f32_parts) {
        part = ws.f32_parts;
        bytes = kF32Parts;
    }
    return lords::launch_prefill_fast(p, part, bytes, ws.zeroed(), (hipStream_t)stream, gate) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int launch_matmul(const lords::MatmulProblem &p, lords_path path, const WsView &ws, void *stream)
{
    hipError_t e;
    if (is_decode(path)) {
        if (use_gemv(p, path)) e = lords::launch_decode_gemv(p, ws.zeroed(), (hipStream_t)stream);
        else if (path == LORDS_PATH_GEMV) return LORDS_ERR_UNSUPPORTED;
        else switch (decode_kind(p)) {
            case kFew: e = lords::launch_decode_mx(p, ws.tickets(), (hipStream_t)stream); break;
            case kFast: e = lords::launch_decode_fast(p, ws.tickets(), (hipStream_t)stream); break;
            default: e = lords::launch_decode(p, ws.scratch(), (hipStream_t)stream);
        }
    } else {
        if (lords::prefill_fast_supported(p)) return launch_large(p, ws, stream);
        e = lords::launch_prefill(p, (hipStream_t)stream);
    }
    return e == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

// The library's own workspace for one checked problem on `path` (already resolved), plus `extra` bytes behind it
// that are left to the caller (*extra_ptr).  `passes`: whether the product may go in two passes.
int plan_workspace(const lords::MatmulProblem &p, lords_path path, size_t extra, void *stream, WsView *ws, void **extra_ptr, bool passes = true)
{
    size_t own = p.f32fact && !is_decode(path) ? kFront : matmul_need(p, path);
    // (bf16 factors: 256-token tiles of one wave per SIMD, and parts that meet, ask for more than there need be)
    const bool elastic = !is_decode(path) && !p.f32fact && own > kFront;
    int rc = passes && !is_decode(path) && lords::two_pass_faster(batch_of(p)) ? two_pass_workspace(batch_of(p), extra, stream, ws, &own)
                                                                             : get_workspace(own + extra, stream, ws, elastic);
    if (rc != LORDS_OK && elastic) {
        own = std::min(own, matmul_least(p, path));
        rc = get_workspace(own + extra, stream, ws);
        ws->bytes = own;                                   // (the plan is made for this much: `extra` lies behind it)
    }
    if (rc == LORDS_OK && extra_ptr) *extra_ptr = ws->base + own;
    return rc;
}

int run_matmul(const lords::MatmulProblem &p, lords_path path, void *stream)
{
    path = resolve_path(path, p);
    if (path == LORDS_PATH_GEMV && !use_gemv(p, path)) return LORDS_ERR_UNSUPPORTED;
    WsView ws;
    const int rc = plan_workspace(p, path, 0, stream, &ws, nullptr);
    return rc != LORDS_OK ? rc : launch_matmul(p, path, ws, stream);
}

// Several matrices that each go to the large-M kernel or into two passes; a status, or -1 (nothing launched) to have them one
// by one.  Every matrix is summed as it would be alone.  Together in two passes: none of them, those that alone would take
// them, or with these the ones that alone are summed by whole tiles, whichever the planner expects to be the fastest with one launch of the
// large-M kernel for the others; a launch of its own is 8 us.  (us, by that kernel all / whichever is faster: 11343 rows of four
// matrices, 864 columns, rank 38, 516 tokens 50 / 50, three in two passes and one after them 66; 6144 rows of three, 4096 columns,
// fp32 rank 64, 2048 tokens 701 / 197.)
int run_batched_large(lords::BatchedProblem bp, void *stream)
{
    if (bp.act) return -1;
    const unsigned all = (1u << bp.L) - 1;
    unsigned whole = 0, alone = 0, in_two = 0;
    for (int l = 0; l < bp.L && bp.M > 128; ++l) {
        const lords::MatmulProblem p = lords::matrix_of(bp, l);
        if (!lords::two_pass_supported(batch_of(p))) continue;
        if (lords::two_pass_faster(batch_of(p))) { alone |= 1u << l; bp.whole[l] = true; }
        else if (lords::prefill_fast_workspace_bytes(p, kNoLimit) == 0) whole |= 1u << l;
    }
    whole |= alone;
    auto pick = [&](unsigned set) { return batch_where(bp, [&](int l) { return (set >> l & 1) != 0; }); };
    if (whole) {
        auto cost = [&](unsigned set) {
            const double two = set ? lords::two_pass_cost(pick(set)) : 0.0;
            return set == all ? two : two + lords::large_cost(pick(all & ~set)) + (set ? 8.0 : 0.0);
        };
        double best = 0.95 * cost(0);
        for (unsigned set : {alone, whole}) {
            if (!set || set == in_two) continue;
            const double us = cost(set);
            if (us < best) { best = us; in_two = set; }
        }
    }
    const lords::BatchedProblem twice = pick(in_two), rest = pick(all & ~in_two);
    WsView ws;
    for (int first = 0, end; first < twice.L; first = end) {
        // (as many at a time as the scratch holds a tile of each of: at 36864 columns seven)
        lords::BatchedProblem group;
        for (end = twice.L; end > first; --end) {
            group = batch_where(twice, [&](int l) { return l >= first && l < end; });
            if (lords::two_pass_supported(group)) break;
        }
        if (end == first) return LORDS_ERR_UNSUPPORTED;        // (not reached: each of them alone is supported)
        size_t own;
        const int rc = two_pass_workspace(group, 0, stream, &ws, &own);
        if (rc != LORDS_OK) return rc;
        if (ws.large == WsView::kTwoPass) {
            if (lords::launch_two_pass(group, ws.scratch(), (hipStream_t)stream) != hipSuccess) return LORDS_ERR_LAUNCH;
        } else {
            for (int l = 0; l < group.L; ++l) {
                const int rcl = launch_large(lords::matrix_of(group, l), ws, stream);
                if (rcl != LORDS_OK) return rcl;
            }
        }
    }
    if (rest.L > 0 && lords::prefill_batched_supported(rest) && get_workspace(kFront + lords::prefill_batched_workspace_bytes(rest), stream, &ws, true) == LORDS_OK)
        return lords::launch_prefill_batched(rest, ws.scratch(), ws.zeroed(), (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
    for (int l = 0; l < rest.L; ++l) {
        const int rc = run_matmul(lords::matrix_of(rest, l), LORDS_PATH_AUTO, stream);
        if (rc != LORDS_OK) return rc;
    }
    return LORDS_OK;
}

// Several matrices in ONE launch, if a kernel takes the case: a status, or -1 if none does.
int run_batched(const lords::BatchedProblem &bp, void *stream)
{
    if (lords::decode_gemv_batched_supported(bp)) {
        WsView ws;
        const int rc = get_workspace(kFront, stream, &ws);
        if (rc != LORDS_OK) return rc;
        return lords::launch_decode_gemv_batched(bp, ws.zeroed(), (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
    }
    if (!lords::decode_mx_batched_supported(bp)) {
        // many tokens: the large-M kernel, if every matrix alone would go there (and their scratch is to be had together)
        for (int l = 0; l < bp.L; ++l) {
            if (is_decode(resolve_path(LORDS_PATH_AUTO, lords::matrix_of(bp, l)))) return -1;
        }
        return run_batched_large(bp, stream);
    }
    WsView ws;
    const int rc = get_workspace(lords::kZeroBytes + lords::decode_mx_batched_workspace_bytes(bp), stream, &ws);
    if (rc != LORDS_OK) return rc;
    return lords::launch_decode_mx_batched(bp, ws.tickets(), (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

// ---- a gate/up pair: matrices 0 and 1 of `bp`, H = Y[0] ----
lords::MatmulProblem gate_up_matrix(const lords::BatchedProblem &bp, int l, void *Y, bool f32out)
{
    return lords::MatmulProblem{bp.X, bp.codes[l], bp.codebook, bp.B[l], bp.A[l], Y, bp.M, bp.N[l], bp.K, bp.r, bp.bits, bp.f32fact, f32out};
}

// Whether the pair's `M` tokens go to the large-M kernel, whose up product multiplies by the gate's silu where it is stored.
bool gate_up_large(lords::BatchedProblem bp, int M)
{
    bp.M = M;
    const lords::MatmulProblem p = gate_up_matrix(bp, 0, nullptr, true);
    return !is_decode(resolve_path(LORDS_PATH_AUTO, p)) && lords::prefill_fast_supported(p);
}

// Tokens to take at once of `left`: 1024 where both products are written to memory, 2048 where the gate alone is (no more
// memory than that).  A few tokens beyond 1024 are not worth tiles of 256 of their own.
//   Up to 16 go to the few-token kernel where it serves the pair in one launch and the layer is not a small one (us, 1025
//   tokens in one piece / cut: 14336 x 4096, 4 bits, rank 32 334 / 262, 11008 x 4096, 3 bits, rank 48 304 / 290, 4096 x 4096
//   133 / 122; 512 x 512 37 / 42).
//   Up to 128, which have tiles of their own size, where the planner sees a twentieth and the second launch's 8 us to be
//   gained (1056 tokens of 14336 x 4096 335 / 304, of 28672 x 4096 622 / 582; not 8192 x 4096, rank 16, 209 / 224).
int gate_up_tokens(lords::BatchedProblem bp, int left)
{
    if (left <= 1024) return left;
    if (!gate_up_large(bp, left)) return 1024;
    if (left >= 2048) return 2048;
    const int rest = left - 1024;
    if (rest <= 16) {
        bp.M = rest;
        const bool few = lords::decode_gemv_batched_supported(bp) || lords::decode_mx_batched_supported(bp);
        return few && (long)bp.N[0] * bp.K >= (4L << 20) ? 1024 : left;
    }
    if (rest > 128) return left;
    lords::MatmulProblem p = gate_up_matrix(bp, 0, nullptr, true);
    auto cost = [&](int M) { p.M = M; return lords::prefill_fast_cost(p); };
    return cost(1024) + cost(rest) + 8.0 < 0.95 * cost(left) ? 1024 : left;
}

// The pair in two passes, all tokens at once: the gate's sums never leave the registers.  Without the scratch: both products by
// whole tiles, the gate's in memory, 2048 tokens at a time or, where there is no room for so many, 1024.
int run_gate_up_two_pass(const lords::BatchedProblem &bp, void *stream)
{
    WsView ws;
    size_t own;
    int rc = two_pass_workspace(bp, 0, stream, &ws, &own);
    if (rc == LORDS_OK && ws.large == WsView::kTwoPass)
        return lords::launch_two_pass(bp, ws.scratch(), (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
    int step = bp.M < 2048 ? bp.M : 2048;
    auto gate_room = [&](bool optional) {                  // (the gate is read four columns at a time)
        return get_workspace(kFront + (size_t)step * bp.N[0] * sizeof(float) + 16, stream, &ws, optional);
    };
    rc = gate_room(step > 1024);
    if (rc != LORDS_OK && step > 1024) {
        step = 1024;
        rc = gate_room(false);
    }
    ws.large = WsView::kWhole;
    for (int m0 = 0; m0 < bp.M && rc == LORDS_OK; m0 += step) {
        lords::BatchedProblem part = bp;
        part.M = bp.M - m0 < step ? bp.M - m0 : step;
        part.X = (const unsigned char *)bp.X + (size_t)m0 * bp.K * 2;
        float *G = (float *)ws.scratch();
        rc = launch_large(gate_up_matrix(part, 0, G, true), ws, stream);
        if (rc != LORDS_OK) break;
        void *H = (unsigned char *)bp.Y[0] + (size_t)m0 * bp.N[0] * (bp.f32out ? 4 : 2);
        rc = launch_large(gate_up_matrix(part, 1, H, bp.f32out), ws, stream, G);
    }
    return rc;
}

// The pair for all bp.M tokens (at most what gate_up_tokens says).  One launch up to 16 tokens where a kernel takes it.
// Otherwise the gate's product goes to the workspace in fp32.  The large-M kernel multiplies by its silu where it stores the
// up product; the general kernels write the up product beside it, and an element-wise pass follows.  The arithmetic is the
// same: fp32 sums, silu(gate) * up in fp32, one rounding.  The seven layers of a block of 4096 / 14336 columns at 2048
// tokens, 4 bits, rank 32: 975 -> 952 us (the element-wise launch took 22 us per 1024 tokens; the gate is now read back by
// the up product's epilogue).
int run_gate_up(const lords::BatchedProblem &bp, void *stream)
{
    const int one = run_batched(bp, stream);
    if (one >= 0) return one;
    const bool fused = gate_up_large(bp, bp.M);
    const size_t count = (size_t)bp.M * bp.N[0], tmp_bytes = (fused ? 1 : 2) * count * sizeof(float) + 16;   // (the gate is read four columns at a time)
    lords::MatmulProblem pg = gate_up_matrix(bp, 0, nullptr, true);
    const lords_path path = resolve_path(LORDS_PATH_AUTO, pg);
    WsView ws;
    void *tmp = nullptr;
    int rc = plan_workspace(pg, path, tmp_bytes, stream, &ws, &tmp, false);
    if (rc != LORDS_OK) return rc;
    float *G = (float *)tmp, *U = G + count;
    pg.Y = G;
    rc = launch_matmul(pg, path, ws, stream);
    if (rc != LORDS_OK) return rc;
    if (fused) return launch_large(gate_up_matrix(bp, 1, bp.Y[0], bp.f32out), ws, stream, G);
    rc = launch_matmul(gate_up_matrix(bp, 1, U, true), path, ws, stream);
    if (rc != LORDS_OK) return rc;
    return lords::launch_silu_mul(G, U, bp.Y[0], (long)count, bp.f32out, (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

// ---- the entry point that allocates nothing: its scratch is this array, one copy per GPU ----
constexpr size_t kStaticBytes = (size_t)24 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];
unsigned char *g_static_ptr[kMaxDevices] = {};
std::mutex g_static_mutex;

int static_workspace(WsView *out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LORDS_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        // the array's name is a host-side stand-in: its device address on THIS GPU is asked for once
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LORDS_ERR_LAUNCH;
        g_static_ptr[dev] = (unsigned char *)ptr;
    }
    out->base = g_static_ptr[dev];
    out->bytes = kStaticBytes;
    return LORDS_OK;
}

inline bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }
inline bool bad_bits(int bits) { return bits != 2 && bits != 3 && bits != 4; }
inline bool bad_dtype(int d) { return d != LORDS_BF16 && d != LORDS_F32; }
inline bool bad_nk(int N, int K) { return N < 1 || K < 32 || (K % 32) != 0; }
inline bool bad_path(int p) { return p < LORDS_PATH_AUTO || p > LORDS_PATH_SMALLM; }

}  // namespace

extern "C" {

int lords_version(void) { return kVersion; }

const char *lords_status_string(int status)
{
    switch (status) {
        case LORDS_OK: return "ok";
        case LORDS_ERR_NULL: return "a required pointer is NULL";
        case LORDS_ERR_BITS: return "bits must be 2, 3 or 4";
        case LORDS_ERR_SHAPE: return "bad shape: need N >= 1, r >= 1, M >= 0, K a positive multiple of 32";
        case LORDS_ERR_ALIGN: return "a pointer is not 16-byte aligned";
        case LORDS_ERR_DTYPE: return "unknown dtype or path value";
        case LORDS_ERR_LAUNCH: return "the HIP runtime refused a launch or an allocation";
        case LORDS_ERR_UNSUPPORTED: return "this shape is not supported by the requested path";
        case LORDS_ERR_WORKSPACE: return "the workspace is missing or too small";
        default: return "unknown status";
    }
}

size_t lords_row_bytes(int K, int bits)
{
    if (bad_bits(bits) || K < 32 || (K % 32) != 0) return 0;
    return (size_t)K / 8 * (size_t)bits;
}

long lords_equivalent_rank(long N, long K, long group)
{
    if (N < 1 || K < 1 || group < 1) return -1;
    const long long num = (long long)N * (long long)K;
    const long long den = (long long)group * ((long long)N + (long long)K);
    return (long)(num / den);
}

int lords_mixed_schedule(int n_layers, double fraction_first, int bits_first, int bits_rest,
                         int *layer_bits, double *avg_bits)
{
    if (!layer_bits) return LORDS_ERR_NULL;
    if (bad_bits(bits_first) || bad_bits(bits_rest)) return LORDS_ERR_BITS;
    if (n_layers < 1 || !(fraction_first >= 0.0)) return LORDS_ERR_SHAPE;
    const double x = fraction_first * (double)n_layers + 0.5;
    const int n_first = x >= (double)n_layers ? n_layers : (int)x;      // x >= 0: truncation is the floor
    long sum = 0;
    for (int l = 0; l < n_layers; ++l) {
        layer_bits[l] = l < n_first ? bits_first : bits_rest;
        sum += layer_bits[l];
    }
    if (avg_bits) *avg_bits = (double)sum / (double)n_layers;
    return LORDS_OK;
}

int lords_unpack(const void *codes, uint8_t *idx, int N, int K, int bits, void *stream)
{
    if (!codes || !idx) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K)) return LORDS_ERR_SHAPE;
    if (misaligned(codes) || misaligned(idx)) return LORDS_ERR_ALIGN;
    return lords::launch_unpack(codes, idx, N, K, bits, (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int lords_dequant(const void *codes, const float *codebook, const void *B, const void *A, void *W,
                  int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype w_dtype, void *stream)
{
    if (!codes || !codebook || !B || !A || !W) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || r < 1) return LORDS_ERR_SHAPE;
    if (misaligned(codes) || misaligned(codebook) || misaligned(B) || misaligned(A) || misaligned(W)) return LORDS_ERR_ALIGN;
    if (bad_dtype((int)factor_dtype) || bad_dtype((int)w_dtype)) return LORDS_ERR_DTYPE;
    return lords::launch_dequant(codes, codebook, B, A, W, N, K, r, bits, factor_dtype == LORDS_F32,
                                 w_dtype == LORDS_F32, (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int lords_quantize(const void *W, const float *codebook, const void *B, const void *A, void *codes,
                   int N, int K, int r, int bits, lords_dtype w_dtype, lords_dtype factor_dtype, void *stream)
{
    if (!W || !codebook || !B || !A || !codes) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || r < 1) return LORDS_ERR_SHAPE;
    if (misaligned(W) || misaligned(codebook) || misaligned(B) || misaligned(A) || misaligned(codes)) return LORDS_ERR_ALIGN;
    if (bad_dtype((int)w_dtype) || bad_dtype((int)factor_dtype)) return LORDS_ERR_DTYPE;
    return lords::launch_quantize(W, codebook, B, A, codes, N, K, r, bits, w_dtype == LORDS_F32,
                                  factor_dtype == LORDS_F32, (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int lords_block_init(const void *W, const float *codebook, void *B, void *A,
                     int N, int K, int r, int bits, lords_dtype w_dtype, lords_dtype factor_dtype, void *stream)
{
    if (!W || !codebook || !B || !A) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || r < 1 || (K % r) != 0) return LORDS_ERR_SHAPE;
    if (misaligned(W) || misaligned(codebook) || misaligned(B) || misaligned(A)) return LORDS_ERR_ALIGN;
    if (bad_dtype((int)w_dtype) || bad_dtype((int)factor_dtype)) return LORDS_ERR_DTYPE;
    return lords::launch_block_init(W, codebook, B, A, N, K, r, bits, w_dtype == LORDS_F32,
                                    factor_dtype == LORDS_F32, (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int lords_matmul_ex(const void *X, const void *codes, const float *codebook, const void *B, const void *A, void *Y,
                    int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype y_dtype,
                    void *stream, lords_path path)
{
    if (!X || !codes || !codebook || !B || !A || !Y) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || r < 1 || M < 0) return LORDS_ERR_SHAPE;
    if (misaligned(X) || misaligned(codes) || misaligned(codebook) || misaligned(B) || misaligned(A) || misaligned(Y))
        return LORDS_ERR_ALIGN;
    if (bad_dtype((int)factor_dtype) || bad_dtype((int)y_dtype)) return LORDS_ERR_DTYPE;
    if (bad_path((int)path)) return LORDS_ERR_DTYPE;
    if (M == 0) return LORDS_OK;
    const bool f32fact = factor_dtype == LORDS_F32;
    if (!lords::fused_rank_supported(r, f32fact)) return LORDS_ERR_UNSUPPORTED;

    lords::MatmulProblem p{X, codes, codebook, B, A, Y, M, N, K, r, bits, f32fact, y_dtype == LORDS_F32};
    return run_matmul(p, path, stream);
}

size_t lords_workspace_zero_bytes(void) { return kFront; }

size_t lords_workspace_bytes(int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_path path)
{
    if (bad_bits(bits) || bad_nk(N, K) || r < 1 || M < 0 || bad_dtype((int)factor_dtype) || bad_path((int)path)) return 0;
    const bool f32fact = factor_dtype == LORDS_F32;
    if (!lords::fused_rank_supported(r, f32fact)) return 0;
    if (M == 0) return kFront;
    lords::MatmulProblem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, M, N, K, r, bits, f32fact, true};
    return matmul_need(p, resolve_path(path, p));
}

namespace {
int matmul_in(const void *X, const void *codes, const float *codebook, const void *B, const void *A, void *Y,
              int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype y_dtype, void *stream,
              lords_path path, const WsView &ws, bool ws_given, bool tiled = false)
{
    if (!X || !codes || !codebook || !B || !A || !Y) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || r < 1 || M < 0) return LORDS_ERR_SHAPE;
    if (misaligned(X) || misaligned(codes) || misaligned(codebook) || misaligned(B) || misaligned(A) || misaligned(Y))
        return LORDS_ERR_ALIGN;
    if (ws_given && (reinterpret_cast<uintptr_t>(ws.base) & 255u) != 0) return LORDS_ERR_ALIGN;
    if (bad_dtype((int)factor_dtype) || bad_dtype((int)y_dtype)) return LORDS_ERR_DTYPE;
    if (bad_path((int)path)) return LORDS_ERR_DTYPE;
    if (M == 0) return LORDS_OK;
    const bool f32fact = factor_dtype == LORDS_F32;
    if (!lords::fused_rank_supported(r, f32fact)) return LORDS_ERR_UNSUPPORTED;
    lords::MatmulProblem p{X, codes, codebook, B, A, Y, M, N, K, r, bits, f32fact, y_dtype == LORDS_F32};
    p.tiled = tiled;
    path = resolve_path(path, p);
    if (path == LORDS_PATH_GEMV && !use_gemv(p, path)) return LORDS_ERR_UNSUPPORTED;
    if (tiled) {
        // the slab-tile layout is read by the one-/two-token, the few-token and the large-M kernel only
        const bool ok = is_decode(path) ? (use_gemv(p, path) || decode_kind(p) == kFew) : lords::prefill_fast_supported(p);
        if (!ok) return LORDS_ERR_UNSUPPORTED;
    }
    // (a caller's workspace must have the size the query gives, or the least that the large-M kernel can do with; the static
    //  one is used as far as it goes, and so is a caller's for a large-M product with fp32 factors, whose whole-tile form
    //  needs the front only)
    const bool elastic = !ws_given || (f32fact && !is_decode(path));
    if (!ws.base || ws.bytes < (elastic ? matmul_need(p, path, ws.bytes) : matmul_least(p, path))) return LORDS_ERR_WORKSPACE;
    return launch_matmul(p, path, ws, stream);
}
}  // namespace

int lords_matmul_ws(const void *X, const void *codes, const float *codebook, const void *B, const void *A, void *Y,
                    int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype y_dtype,
                    void *stream, lords_path path, void *workspace, size_t workspace_bytes)
{
    WsView ws;
    ws.base = (unsigned char *)workspace;
    ws.bytes = workspace_bytes;
    return matmul_in(X, codes, codebook, B, A, Y, M, N, K, r, bits, factor_dtype, y_dtype, stream, path, ws, true);
}

size_t lords_repack_bytes(int N, int K, int bits)
{
    if (bad_bits(bits) || bad_nk(N, K)) return 0;
    return (size_t)((N + 15) / 16) * (size_t)((K + 127) / 128) * 256u * (size_t)bits;
}

int lords_repack(const void *codes, void *codes_tiled, int N, int K, int bits, void *stream)
{
    if (!codes || !codes_tiled) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K)) return LORDS_ERR_SHAPE;
    if (misaligned(codes) || misaligned(codes_tiled)) return LORDS_ERR_ALIGN;
    return lords::launch_repack(codes, codes_tiled, N, K, bits, (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int lords_matmul_repacked(const void *X, const void *codes_tiled, const float *codebook, const void *B, const void *A, void *Y,
                          int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype y_dtype,
                          void *stream, lords_path path)
{
    // argument checks first (no workspace is touched for a bad call), then the library's own workspace
    WsView none;
    const int rc0 = matmul_in(X, codes_tiled, codebook, B, A, Y, M, N, K, r, bits, factor_dtype, y_dtype, stream, path, none, false, true);
    if (rc0 != LORDS_ERR_WORKSPACE) return rc0;          // LORDS_OK only for M == 0
    const bool f32fact = factor_dtype == LORDS_F32;
    lords::MatmulProblem p{X, codes_tiled, codebook, B, A, Y, M, N, K, r, bits, f32fact, y_dtype == LORDS_F32};
    p.tiled = true;
    WsView ws;
    const int rc = plan_workspace(p, resolve_path(path, p), 0, stream, &ws, nullptr);
    if (rc != LORDS_OK) return rc;
    return matmul_in(X, codes_tiled, codebook, B, A, Y, M, N, K, r, bits, factor_dtype, y_dtype, stream, path, ws, false, true);
}

size_t lords_noalloc_limit(void) { return kStaticBytes; }

int lords_matmul_noalloc(const void *X, const void *codes, const float *codebook, const void *B, const void *A, void *Y,
                         int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype y_dtype, void *stream)
{
    WsView ws;
    const int rc = static_workspace(&ws);
    if (rc != LORDS_OK) return rc;
    return matmul_in(X, codes, codebook, B, A, Y, M, N, K, r, bits, factor_dtype, y_dtype, stream, LORDS_PATH_AUTO, ws, false);
}

int lords_matmul_batched(const void *X, const void *const *codes, const float *codebook, const void *const *B,
                         const void *const *A, void *const *Y, const int *N, int L, int M, int K, int r, int bits,
                         lords_dtype factor_dtype, lords_dtype y_dtype, void *stream)
{
    if (!X || !codes || !codebook || !B || !A || !Y || !N) return LORDS_ERR_NULL;
    if (L < 1 || L > lords::kMaxBatch) return LORDS_ERR_SHAPE;
    for (int l = 0; l < L; ++l)
        if (!codes[l] || !B[l] || !A[l] || !Y[l]) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (K < 32 || (K % 32) != 0 || r < 1 || M < 0) return LORDS_ERR_SHAPE;
    for (int l = 0; l < L; ++l)
        if (N[l] < 1) return LORDS_ERR_SHAPE;
    if (misaligned(X) || misaligned(codebook)) return LORDS_ERR_ALIGN;
    for (int l = 0; l < L; ++l)
        if (misaligned(codes[l]) || misaligned(B[l]) || misaligned(A[l]) || misaligned(Y[l])) return LORDS_ERR_ALIGN;
    if (bad_dtype((int)factor_dtype) || bad_dtype((int)y_dtype)) return LORDS_ERR_DTYPE;
    if (M == 0) return LORDS_OK;
    const bool f32fact = factor_dtype == LORDS_F32;
    if (!lords::fused_rank_supported(r, f32fact)) return LORDS_ERR_UNSUPPORTED;

    lords::BatchedProblem bp;
    bp.X = X; bp.codebook = codebook;
    for (int l = 0; l < lords::kMaxBatch; ++l) {
        const int s = l < L ? l : 0;
        bp.codes[l] = codes[s]; bp.B[l] = B[s]; bp.A[l] = A[s]; bp.Y[l] = Y[s]; bp.N[l] = N[s];
    }
    bp.L = L; bp.M = M; bp.K = K; bp.r = r; bp.bits = bits;
    bp.f32fact = f32fact; bp.f32out = y_dtype == LORDS_F32; bp.act = false;
    if (L > 1) {
        const int rc = run_batched(bp, stream);
        if (rc >= 0) return rc;
    }
    // a case no one-launch kernel takes: matrix by matrix
    for (int l = 0; l < L; ++l) {
        lords::MatmulProblem p{X, codes[l], codebook, B[l], A[l], Y[l], M, N[l], K, r, bits, f32fact, y_dtype == LORDS_F32};
        const int rc = run_matmul(p, LORDS_PATH_AUTO, stream);
        if (rc != LORDS_OK) return rc;
    }
    return LORDS_OK;
}

int lords_gate_up(const void *X, const void *codes_gate, const void *B_gate, const void *A_gate,
                  const void *codes_up, const void *B_up, const void *A_up, const float *codebook, void *H,
                  int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype h_dtype, void *stream)
{
    if (!X || !codes_gate || !B_gate || !A_gate || !codes_up || !B_up || !A_up || !codebook || !H) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || r < 1 || M < 0) return LORDS_ERR_SHAPE;
    if (misaligned(X) || misaligned(codes_gate) || misaligned(B_gate) || misaligned(A_gate) || misaligned(codes_up) ||
        misaligned(B_up) || misaligned(A_up) || misaligned(codebook) || misaligned(H))
        return LORDS_ERR_ALIGN;
    if (bad_dtype((int)factor_dtype) || bad_dtype((int)h_dtype)) return LORDS_ERR_DTYPE;
    if (M == 0) return LORDS_OK;
    const bool f32fact = factor_dtype == LORDS_F32, f32out = h_dtype == LORDS_F32;
    if (!lords::fused_rank_supported(r, f32fact)) return LORDS_ERR_UNSUPPORTED;

    lords::BatchedProblem bp;
    bp.X = X; bp.codebook = codebook;
    for (int l = 0; l < lords::kMaxBatch; ++l) {
        const bool up = l == 1;
        bp.codes[l] = up ? codes_up : codes_gate; bp.B[l] = up ? B_up : B_gate; bp.A[l] = up ? A_up : A_gate;
        bp.Y[l] = H; bp.N[l] = N;
    }
    bp.L = 2; bp.M = M; bp.K = K; bp.r = r; bp.bits = bits;
    bp.f32fact = f32fact; bp.f32out = f32out; bp.act = true;
    if (gate_up_large(bp, M) && lords::two_pass_faster(bp)) return run_gate_up_two_pass(bp, stream);
    for (int m0 = 0, mc; m0 < M; m0 += mc) {
        mc = gate_up_tokens(bp, M - m0);
        bp.M = mc;
        bp.X = (const unsigned char *)X + (size_t)m0 * K * 2;
        bp.Y[0] = bp.Y[1] = (unsigned char *)H + (size_t)m0 * N * (f32out ? 4 : 2);
        const int rc = run_gate_up(bp, stream);
        if (rc != LORDS_OK) return rc;
    }
    return LORDS_OK;
}

int lords_transpose_codes(const void *codes, void *codes_t, int N, int K, int bits, void *stream)
{
    if (!codes || !codes_t) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || (N % 32) != 0) return LORDS_ERR_SHAPE;
    if (misaligned(codes) || misaligned(codes_t)) return LORDS_ERR_ALIGN;
    return lords::launch_transpose_codes(codes, codes_t, N, K, bits, (hipStream_t)stream) == hipSuccess ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int lords_backward_input(const void *dY, const void *codes_t, const float *codebook, const void *B, const void *A, void *dX,
                         int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype dx_dtype, void *stream)
{
    if (!dY || !codes_t || !codebook || !B || !A || !dX) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || (N % 32) != 0 || r < 1 || M < 0) return LORDS_ERR_SHAPE;
    if (misaligned(dY) || misaligned(codes_t) || misaligned(codebook) || misaligned(B) || misaligned(A) || misaligned(dX))
        return LORDS_ERR_ALIGN;
    if (bad_dtype((int)factor_dtype) || bad_dtype((int)dx_dtype)) return LORDS_ERR_DTYPE;
    if (M == 0) return LORDS_OK;
    const bool f32fact = factor_dtype == LORDS_F32;
    if (!lords::fused_rank_supported(r, f32fact)) return LORDS_ERR_UNSUPPORTED;
    // The transposed layer: rows = the K in-features, columns = the N out-features, factors A^T (K x r)
    // and B^T (r x N); its forward product applied to dY is dX.
    const size_t esz = f32fact ? 4 : 2;
    const size_t at_bytes = ((size_t)K * r * esz + 255) & ~(size_t)255, bt_bytes = ((size_t)r * N * esz + 255) & ~(size_t)255;
    lords::MatmulProblem p{dY, codes_t, codebook, nullptr, nullptr, dX, M, K, N, r, bits, f32fact, dx_dtype == LORDS_F32};
    const lords_path path = resolve_path(LORDS_PATH_AUTO, p);
    WsView ws;
    void *extra = nullptr;
    const int rc = plan_workspace(p, path, at_bytes + bt_bytes, stream, &ws, &extra);
    if (rc != LORDS_OK) return rc;
    void *At = extra, *Bt = (unsigned char *)extra + at_bytes;
    if (lords::launch_transpose_factors(A, At, B, Bt, N, K, r, f32fact, (hipStream_t)stream) != hipSuccess) return LORDS_ERR_LAUNCH;
    p.B = At;
    p.A = Bt;
    return launch_matmul(p, path, ws, stream);
}

int lords_backward_factors(const void *dY, const void *X, const void *codes, const float *codebook, const void *B,
                           const void *A, float *dB, float *dA, int M, int N, int K, int r, int bits,
                           lords_dtype factor_dtype, void *stream)
{
    if (!dY || !X || !codes || !codebook || !B || !A || !dB || !dA) return LORDS_ERR_NULL;
    if (bad_bits(bits)) return LORDS_ERR_BITS;
    if (bad_nk(N, K) || r < 1 || M < 0) return LORDS_ERR_SHAPE;
    if (misaligned(dY) || misaligned(X) || misaligned(codes) || misaligned(codebook) || misaligned(B) || misaligned(A) ||
        misaligned(dB) || misaligned(dA))
        return LORDS_ERR_ALIGN;
    if (bad_dtype((int)factor_dtype)) return LORDS_ERR_DTYPE;
    if (!lords::factor_grad_supported(N, K, r)) return LORDS_ERR_UNSUPPORTED;
    WsView ws;
    const int rc = get_workspace(kFront + lords::factor_grad_workspace_bytes(N, K, r), stream, &ws);
    if (rc != LORDS_OK) return rc;
    return lords::launch_factor_grad(dY, X, codes, codebook, B, A, dB, dA, M, N, K, r, bits, factor_dtype == LORDS_F32,
                                     ws.scratch(), (hipStream_t)stream) == hipSuccess
               ? LORDS_OK : LORDS_ERR_LAUNCH;
}

int lords_matmul(const void *X, const void *codes, const float *codebook, const void *B, const void *A, void *Y,
                 int M, int N, int K, int r, int bits, lords_dtype factor_dtype, lords_dtype y_dtype, void *stream)
{
    return lords_matmul_ex(X, codes, codebook, B, A, Y, M, N, K, r, bits, factor_dtype, y_dtype, stream, LORDS_PATH_AUTO);
}

}  // extern "C"
