// The library's planner for tests: problems are put together by the library's own header, so that its structures are never
// copied by hand.
#include "../paper_2601_22716_amd/csrc/lords_launch.h"

namespace {
lords::BatchedProblem batched(const int *N, int L, int M, int K, int r, int bits, int f32, int act)
{
    lords::BatchedProblem p{};
    for (int l = 0; l < L; ++l) p.N[l] = N[l];
    p.L = L; p.M = M; p.K = K; p.r = r; p.bits = bits;
    p.f32fact = f32 != 0; p.f32out = true; p.act = act != 0;
    return p;
}
lords::MatmulProblem single(int M, int N, int K, int r, int bits, int f32)
{
    lords::MatmulProblem p{};
    p.M = M; p.N = N; p.K = K; p.r = r; p.bits = bits;
    p.f32fact = f32 != 0; p.f32out = true;
    return p;
}
}  // namespace

extern "C" {
int two_pass_faster(const int *N, int L, int M, int K, int r, int bits, int f32, int act) { return lords::two_pass_faster(batched(N, L, M, K, r, bits, f32, act)); }
int two_pass_supported(const int *N, int L, int M, int K, int r, int bits, int f32, int act) { return lords::two_pass_supported(batched(N, L, M, K, r, bits, f32, act)); }
size_t two_pass_workspace_bytes(const int *N, int L, int M, int K, int r, int bits, int f32, int act) { return lords::two_pass_workspace_bytes(batched(N, L, M, K, r, bits, f32, act)); }
size_t prefill_workspace_bytes(int M, int N, int K, int r, int bits, int f32) { return lords::prefill_fast_workspace_bytes(single(M, N, K, r, bits, f32), ~(size_t)0); }
size_t prefill_least_workspace_bytes(int M, int N, int K, int r, int bits, int f32) { return lords::prefill_least_workspace_bytes(single(M, N, K, r, bits, f32)); }
void prefill_cut(int M, int N, int K, int r, int bits, int f32, int *tokens_rows_parts)
{
    const lords::PrefillCut cut = lords::prefill_cut(single(M, N, K, r, bits, f32), ~(size_t)0);
    tokens_rows_parts[0] = cut.tokens; tokens_rows_parts[1] = cut.rows; tokens_rows_parts[2] = cut.meet;
}
void prefill_batched_cut(const int *N, int L, int M, int K, int r, int bits, int f32, int l, int *tokens_rows_parts_walk)
{
    const lords::PrefillCut cut = lords::prefill_batched_cut(batched(N, L, M, K, r, bits, f32, 0), l);
    tokens_rows_parts_walk[0] = cut.tokens; tokens_rows_parts_walk[1] = cut.rows; tokens_rows_parts_walk[2] = cut.meet; tokens_rows_parts_walk[3] = cut.walk;
}
double prefill_batched_cost(const int *N, int L, int M, int K, int r, int bits, int f32) { return lords::prefill_batched_cost(batched(N, L, M, K, r, bits, f32, 0)); }
size_t prefill_batched_workspace_bytes(const int *N, int L, int M, int K, int r, int bits, int f32) { return lords::prefill_batched_workspace_bytes(batched(N, L, M, K, r, bits, f32, 0)); }
int prefill_wide_taken(int M, int N, int K, int r, int bits, int f32) { return lords::prefill_wide_taken(single(M, N, K, r, bits, f32), ~(size_t)0); }
// The large-M kernel itself, with a say in how long a workgroup waits for the parts of others; scratch of the size above.
int launch_large(const void *X, const void *codes, const float *codebook, const void *B, const void *A, void *Y, const float *gate, int M, int N, int K,
                 int r, int bits, int f32, int f32out, void *part, size_t part_bytes, void *zeroed, void *stream, int polls)
{
    lords::MatmulProblem p = single(M, N, K, r, bits, f32);
    p.X = X; p.codes = codes; p.codebook = codebook; p.B = B; p.A = A; p.Y = Y; p.f32out = f32out != 0;
    return (int)lords::launch_prefill_fast(p, part, part_bytes, zeroed, (hipStream_t)stream, gate, polls);
}
int launch_large_batched(const void *X, const void *const *codes, const float *codebook, const void *const *B, const void *const *A, void *const *Y, const int *N,
                         int L, int M, int K, int r, int bits, int f32, int f32out, void *part, void *zeroed, void *stream, int polls)
{
    lords::BatchedProblem p = batched(N, L, M, K, r, bits, f32, 0);
    p.X = X; p.codebook = codebook; p.f32out = f32out != 0;
    for (int l = 0; l < L; ++l) { p.codes[l] = codes[l]; p.B[l] = B[l]; p.A[l] = A[l]; p.Y[l] = Y[l]; }
    return (int)lords::launch_prefill_batched(p, part, zeroed, (hipStream_t)stream, polls);
}
}
