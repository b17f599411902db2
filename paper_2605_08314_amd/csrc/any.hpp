// Products of whole-number sizes at any alignment (rows of any number above the decode kernels' 32): launch descriptors and
// host planners of the any-size tile kernels.
#pragma once
#include "lr_common.hpp"

namespace lr {

// What a launch writes: ANY_T fp32 rows (rank space, or partial sums of a K chunk), ANY_GATEUP fp32 hidden rows
// SiLU(g + b_g) * (u + b_u) of two products, ANY_OUT the result in the call's element type, + bias, to C and / or a cache.
enum { ANY_T = 0, ANY_GATEUP = 1, ANY_OUT = 2 };
constexpr int kMaxAny = 8;
constexpr int kAnyTile = 128, kAnyStep = 32;      // rows and columns of a bf16 tile, k of a step

// C[M, N] = A[M, K] * B[K, N]; A has row stride lda, B is contiguous row-major.
struct AnyProb {
    const void* A;  int64_t lda;  const void* B;  int K;
    const void* A2; int64_t lda2; const void* B2; int K2;      // ANY_GATEUP: the up-branch product
    int N;
    void* C; int64_t ldc;
    const void* bias; const void* bias2;
    void* cache; const int32_t* pos; int S_max; int T;
    int splits, kchunk; int64_t split_stride;                  // ANY_T: K chunks, rows per chunk, floats between the chunks' results
    int tiles_n, tile_begin;
};
struct AnyArgs { AnyProb p[kMaxAny]; int nprob, M, tiles_m, first, count; };      // a launch takes tiles [first, first + count)
// Tiles of a launch: a grid has fewer than 2^32 threads and a workgroup up to 512.  More tiles (2^27 rows of a narrow fp32 result)
// run as several launches.
constexpr int kAnyLaunchTiles = 1 << 22;

// Rows, K and N the kernels index with 32-bit numbers
bool any_rows_ok(int64_t M);
bool any_factor_ok(int64_t K, int64_t N);
// One launch of the products of `a` (fills in the tiling).  a_f32 (bf16 calls): A is fp32 rank-space or hidden rows.
int any_launch_bf16(AnyArgs& a, bool a_f32, int epi, hipStream_t s);
int any_launch_f32(AnyArgs& a, int epi, hipStream_t s);
// dst[i] = sum of part[i + c * stride] over chunks c < splits, in order
int any_reduce(const float* part, float* dst, int64_t n, int splits, int64_t stride, hipStream_t s);
// The calls of include/lowrank.h.  t_only: no workspace, only this area of M * r floats.  base_of / t_off / R as in prefill_qkv.
int any_qkv(const void* x, const void* const* U, const void* const* V, const void* const* bias,
            void* const* out, const int64_t* r, const int64_t* d_out, int n_proj, const int* base_of,
            const int64_t* t_off, int64_t R, int64_t M, int64_t d_in, const lr_kv_target* kv,
            void* ws, size_t ws_bytes, int dtype, hipStream_t s);
int any_linear(const void* x, const void* U, const void* V, const void* bias, void* y,
               int64_t M, int64_t d_in, int64_t r, int64_t d_out, void* ws, size_t ws_bytes, float* t_only, int dtype, hipStream_t s);
int any_mlp(const void* x, const void* U_gu, const void* V_g, const void* V_u, const void* U_d,
            const void* V_d, const void* b_g, const void* b_u, const void* b_d, void* out,
            int64_t M, int64_t d, int64_t ffn, int64_t r_g, int64_t r_u, int64_t r_d,
            void* ws, size_t ws_bytes, int dtype, hipStream_t s);
int any_rank_project(const void* x, const void* U, void* t, int64_t M, int64_t d_in, int64_t r,
                     void* ws, size_t ws_bytes, int dtype, hipStream_t s);

}  // namespace lr
