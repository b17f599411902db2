// fp32 products of any sizes and alignment with fp64 accumulation, on the fp64 matrix cores (v_mfma_f64_16x16x4_f64).
//
// fp32 operands are exact in fp64 and every sum of a call is kept in fp64 until its one rounding, as the generic kernels do.
// Bound by the fp64 rate (79 TFLOP/s, a thirtieth of bf16): a 16-k step of one 16 x 64 block takes 1024 matrix-core cycles for
// 5 KB of operands, so nothing is staged through LDS; a wave loads its operands straight into the layout of the instruction.
//   A  lane (j, g) = (lane % 16, lane / 16) holds 4 consecutive k (16 s + 4 g ..) of row j: one 16-byte load per step
//   B  the same lane holds CPL consecutive columns of rows 16 s + 4 g + t, t = 0 .. 3: four loads of 4 * CPL bytes, 16 lanes side by side
// Instruction (t, b) multiplies k = {16 s + 4 g + t} (any order of k will do, as long as both operands agree on it) and gives
// the columns CPL * j + b.  The eight waves of a workgroup take the steps of a tile in turn, their fp64 partial sums meet in LDS.
// Measured (one thread per output element before): 16 x 512 x 128 x 512 10.9 us per call, bound by the host's two launches
// (66 us); packed MLP of 200 rows, d = 1024, ffn = 2816, ranks 192: 47 us, four launches of 6-18 us (1135 us);
// 4096^4 61 TFLOP/s, where the vendor library's fp64 product reaches 70.
#include "any.hpp"

namespace lr {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

template <int MB, int CPL> struct F32Regs { float a[MB][4]; float b[4][CPL]; };

struct F32Operands {
    const float* A;
    const float* B; int N;            // column n0 of row 0 (uniform)
    int K; int64_t avail;             // elements of B from `B` to the matrix's end
};

// a step that exists as a whole (a tile past the last column reads on into the next row; those columns are never stored)
template <int MB, int CPL>
__device__ __forceinline__ void f32_load(F32Regs<MB, CPL>& r, const F32Operands& o, const int64_t (&arow)[MB], int s, int j, int g) {
    const int k0 = 16 * s;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) __builtin_memcpy(r.a[mb], o.A + arow[mb] + k0, 16);
    const float* b = o.B + (size_t)k0 * (size_t)o.N;
#pragma unroll
    for (int t = 0; t < 4; ++t) __builtin_memcpy(r.b[t], b + ((4 * g + t) * o.N + CPL * j), 4 * CPL);
}
// a step at the end of K or of the matrix: element by element, zero where nothing exists
template <int MB, int CPL>
__device__ __forceinline__ void f32_load_end(F32Regs<MB, CPL>& r, const F32Operands& o, const int64_t (&arow)[MB], int s, int j, int g) {
    const int k0 = 16 * s;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int t = 0; t < 4; ++t) r.a[mb][t] = k0 + 4 * g + t < o.K ? o.A[arow[mb] + k0 + t] : 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int64_t at = (int64_t)(k0 + 4 * g + t) * o.N + CPL * j;
#pragma unroll
        for (int b = 0; b < CPL; ++b) r.b[t][b] = at + b < o.avail ? o.B[at + b] : 0.f;
    }
}

template <int MB, int CPL>
__device__ __forceinline__ void f32_mma(f64x4_t (&acc)[MB][CPL], const F32Regs<MB, CPL>& r) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int b = 0; b < CPL; ++b)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                acc[mb][b] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)r.a[mb][t], (double)r.b[t][b], acc[mb][b], 0, 0, 0);
}

// steps part, part + KW, ... of A B, PF of them in flight (those at the end of the matrix afterwards, one by one)
template <int MB, int CPL, int KW>
__device__ __forceinline__ void f32_product(f64x4_t (&acc)[MB][CPL], const float* A, int64_t lda, const float* B, int N, int K,
                                            int M, int m0, int n0, int part, int j, int g) {
    constexpr int PF = 8 / CPL;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int b = 0; b < CPL; ++b) acc[mb][b] = f64x4_t{0., 0., 0., 0.};
    F32Operands o;
    o.A = A; o.B = B + n0; o.N = N; o.K = K; o.avail = (int64_t)K * N - n0;
    int64_t arow[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        int m = m0 + 16 * mb + j;
        m = m < M ? m : M - 1;                       // rows past the end repeat the last one; never stored
        arow[mb] = (int64_t)m * lda + 4 * g;
    }
    const int ns = (K + 15) >> 4;
    // whole steps: 16 s + 16 <= K, and (16 s + 15) N + 16 CPL elements from the tile's first on exist
    const int64_t fit = o.avail < 16 * CPL ? 0 : ((o.avail - 16 * CPL) / N + 1) >> 4;
    const int nf = fit < (K >> 4) ? (int)fit : K >> 4;
    F32Regs<MB, CPL> r[PF];
#pragma unroll
    for (int p = 0; p < PF; ++p)
        if (part + KW * p < nf) f32_load<MB, CPL>(r[p], o, arow, part + KW * p, j, g);
    for (int s = part; s < nf; s += KW * PF) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            const int sp = s + KW * p;
            if (sp < nf) {
                f32_mma<MB, CPL>(acc, r[p]);
                if (sp + KW * PF < nf) f32_load<MB, CPL>(r[p], o, arow, sp + KW * PF, j, g);
            }
        }
    }
#pragma unroll 1
    for (int s = part; s < ns; s += KW) {
        if (s < nf) continue;
        f32_load_end<MB, CPL>(r[0], o, arow, s, j, g);
        f32_mma<MB, CPL>(acc, r[0]);
    }
}

template <int MB, int CPL, int EPI>
__global__ void __launch_bounds__(512, MB == 1 ? 4 : 2) k_f32_gemm(AnyArgs ga) {
    constexpr int NC = 16 * CPL, NSL = MB * CPL * 4, ITEMS = MB * 256, PER = (ITEMS + 511) / 512;
    constexpr int NMAT = EPI == ANY_GATEUP ? 2 : 1, KW = 8 / NMAT;      // gate/up: waves 0-3 multiply the gate branch, 4-7 the up branch
    __shared__ double red[8 * NSL * 64];
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups go to the 8 XCDs round-robin: each XCD gets a run of tiles, row tiles of one column tile next to each other
    const int per = (ga.count + 7) >> 3;
    const int local = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (local >= ga.count) return;
    const int id = ga.first + local;
    int pi = 0;
#pragma unroll
    for (int i = 1; i < kMaxAny; ++i)
        if (i < ga.nprob && id >= ga.p[i].tile_begin) pi = i;
    const AnyProb& P = ga.p[pi];
    const int rem = id - P.tile_begin, tn = rem / ga.tiles_m, tm = rem - tn * ga.tiles_m;
    const int m0 = tm * 16 * MB, n0 = tn * NC, M = ga.M, N = P.N;

    f64x4_t acc[MB][CPL];
    const bool up = EPI == ANY_GATEUP && wave >= KW;
    f32_product<MB, CPL, KW>(acc, (const float*)(up ? P.A2 : P.A), up ? P.lda2 : P.lda, (const float*)(up ? P.B2 : P.B), N, up ? P.K2 : P.K,
                             M, m0, n0, wave & (KW - 1), j, g);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int b = 0; b < CPL; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) red[(wave * NSL + (mb * CPL + b) * 4 + i) * 64 + lane] = acc[mb][b][i];
    __syncthreads();
    // result register i of lane (j, g) is row g + 4 i, column CPL j + b
    double sum[NMAT][PER][CPL];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int it = tid + 512 * q;
        const int row = it >> 4, jj = it & 15, mb = row >> 4, r16 = row & 15;
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat)
#pragma unroll
            for (int b = 0; b < CPL; ++b) {
                double v = 0.;
                if (it < ITEMS)
                    for (int w = 0; w < KW; ++w) v += red[((mat * KW + w) * NSL + (mb * CPL + b) * 4 + (r16 >> 2)) * 64 + (r16 & 3) * 16 + jj];
                sum[mat][q][b] = v;
            }
    }
    const float* bias = (const float*)P.bias;
    const float* bias2 = (const float*)P.bias2;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int it = tid + 512 * q;
        const int m = m0 + (it >> 4), n = n0 + CPL * (it & 15);
        if (it >= ITEMS || m >= M || n >= N) continue;
        float v[CPL];
#pragma unroll
        for (int b = 0; b < CPL; ++b) {
            double x = sum[0][q][b];
            if (bias && n + b < N) x += (double)bias[n + b];
            if constexpr (EPI == ANY_GATEUP) {
                double u = sum[NMAT - 1][q][b];
                if (bias2 && n + b < N) u += (double)bias2[n + b];
                v[b] = silu_f32((float)x) * (float)u;
            } else v[b] = (float)x;
        }
        auto store = [&](float* d) {
            if (n + CPL <= N) __builtin_memcpy(d, v, 4 * CPL);
            else {
#pragma unroll
                for (int b = 0; b < CPL; ++b) if (n + b < N) d[b] = v[b];
            }
        };
        if (P.C) store((float*)P.C + (size_t)m * (size_t)P.ldc + n);
        if constexpr (EPI == ANY_OUT) {
            if (P.cache) {
                const int bi = m / P.T;
                const int64_t pp = (int64_t)P.pos[bi] + (m - bi * P.T);
                if (pp >= 0 && pp < P.S_max) store((float*)P.cache + ((size_t)bi * (size_t)P.S_max + (size_t)pp) * (size_t)N + n);
            }
        }
    }
}

template <int MB, int CPL>
static int launch_f32(AnyArgs& a, int epi, hipStream_t s) {
    const int rows = 16 * MB, cols = 16 * CPL;
    a.tiles_m = (a.M + rows - 1) / rows;
    int64_t total = 0;
    for (int i = 0; i < a.nprob; ++i) {
        AnyProb& p = a.p[i];
        p.tiles_n = (p.N + cols - 1) / cols; p.tile_begin = (int)total;
        total += (int64_t)a.tiles_m * p.tiles_n;
    }
    if (total <= 0) return LR_OK;
    if (total >= (1ll << 31)) { set_error("too many output tiles"); return LR_ERR_UNSUPPORTED; }
    for (int64_t first = 0; first < total; first += kAnyLaunchTiles) {
        a.first = (int)first;
        a.count = (int)(total - first < kAnyLaunchTiles ? total - first : kAnyLaunchTiles);
        const dim3 grid((unsigned)((a.count + 7) / 8 * 8)), block(512);
        if (epi == ANY_T) hipLaunchKernelGGL((k_f32_gemm<MB, CPL, ANY_T>), grid, block, 0, s, a);
        else if (epi == ANY_GATEUP) {
            if constexpr (MB == 1) hipLaunchKernelGGL((k_f32_gemm<MB, CPL, ANY_GATEUP>), grid, block, 0, s, a);
        } else hipLaunchKernelGGL((k_f32_gemm<MB, CPL, ANY_OUT>), grid, block, 0, s, a);
        const int st = launch_status("fp32 product");
        if (st != LR_OK) return st;
    }
    return LR_OK;
}

int any_launch_f32(AnyArgs& a, int epi, hipStream_t s) {
    // The widest tile that still gives every CU a workgroup: the wider, the fewer widenings of A to fp64 and loads per matrix
    // instruction; two 16-row blocks (B loaded and widened once for both) when even
    // 32 x 64 tiles fill the chip twice (not for gate/up, whose second product would spill)
    auto tiles = [&](int rows, int cols) {
        int64_t t = 0;
        for (int i = 0; i < a.nprob; ++i) t += (int64_t)((a.M + rows - 1) / rows) * ((a.p[i].N + cols - 1) / cols);
        return t;
    };
    if (epi != ANY_GATEUP && tiles(32, 64) >= 512) return launch_f32<2, 4>(a, epi, s);
    if (tiles(16, 64) >= 256) return launch_f32<1, 4>(a, epi, s);
    if (tiles(16, 32) >= 256) return launch_f32<1, 2>(a, epi, s);
    return launch_f32<1, 1>(a, epi, s);
}

}  // namespace lr
