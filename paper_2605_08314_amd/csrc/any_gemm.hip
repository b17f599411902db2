// bf16 products of whole-number sizes at any alignment, more than 32 rows: 128 x 128 tiles on the matrix cores.
//
// The tuned prefill kernel moves both operands global memory -> LDS directly, 16 aligned bytes per lane; rows of odd length
// have no such units.  Here the operands pass through registers instead: global loads of 16 bytes at any 2-byte alignment,
// ds_write into the same swizzled LDS tiles, the same fragment reads (any_gemm shares prefill_device.hpp).  A step is 32 k;
// its loads are issued two steps before they are written to LDS, which is one barrier before they are read; two workgroups
// per CU cover each other's barriers.
//
// Bound by the matrix cores and the register path around them.  Measured: a layer of 1500 rows at d = 4096, ffn = 11008, ranks
// 371 / 755 with its attention 643 us (one thread per output element before: 40.3 ms).
//
// Precision: rank-space and hidden rows stay fp32 between the launches.  Such an operand is cut on its way into LDS into three
// bf16 parts that add up to all its 24 bits and multiplied in three matrix instructions per fragment pair, so that only the
// result is rounded to bf16.  B is read once for all three.  (Two parts keep 16 bits: 4.5e-6 of the result before its rounding,
// where plain fp32 is off by less than 1e-6; the layer above took 568 us with them.)
#include "any.hpp"
#include "decode.hpp"
#include "prefill_device.hpp"

namespace lr {

constexpr int ABM = kAnyTile, ABN = kAnyTile, ABK = kAnyStep;
constexpr int kATile = ABM * ABK * 2, kBTile = ABK * ABN * 2;         // bytes of a bf16 tile in LDS
constexpr int kRest = kATile + kBTile;                                // a stage: A (first part) | B | A second part | A third part
template <bool AF32> constexpr int any_stage_bytes() { return kRest + (AF32 ? 2 * kATile : 0); }

// One thread's share of a step: two 8-k units of A (fp32: 32 bytes each), two 8-column units of B.
template <bool AF32> struct AnyRegs { uint4 a[AF32 ? 4 : 2]; uint4 b[2]; };

struct AnyOperands {
    const char* a[2];            // this thread's A rows at k = 0 of its units
    const bf16_t* B;             // the tile's first column of row 0
    int N;
    int64_t avail;               // elements of B from `B` to the matrix's end
    int K;                       // end of the K range
};

template <bool AF32>
__device__ __forceinline__ void any_load(AnyRegs<AF32>& r, const AnyOperands& o, int k0) {
    const int tid = threadIdx.x;
    const int c = (tid & 3) * 8;
    // uniform: the step lies inside K and its B rows inside the matrix (a tile past the last column reads on into the next
    // row: those columns are never stored)
    if (k0 + ABK <= o.K && (int64_t)(k0 + ABK - 1) * o.N + ABN <= o.avail) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (AF32) {
                const char* p = o.a[j] + (size_t)k0 * 4;
                __builtin_memcpy(&r.a[2 * j], p, 16); __builtin_memcpy(&r.a[2 * j + 1], p + 16, 16);
            } else {
                __builtin_memcpy(&r.a[j], o.a[j] + (size_t)k0 * 2, 16);
            }
        }
        const bf16_t* b = o.B + (size_t)k0 * (size_t)o.N;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lin = j * 256 + tid, kr = lin >> 4, u = lin & 15;
            __builtin_memcpy(&r.b[j], b + (kr * o.N + u * 8), 16);
        }
    } else {
        // element by element, zero where nothing exists (zero on both sides: a stray infinity times zero would be NaN)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (AF32) {
                const float* p = reinterpret_cast<const float*>(o.a[j]) + k0;
                uint32_t e[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) e[i] = k0 + c + i < o.K ? __float_as_uint(p[i]) : 0u;
                r.a[2 * j] = make_uint4(e[0], e[1], e[2], e[3]); r.a[2 * j + 1] = make_uint4(e[4], e[5], e[6], e[7]);
            } else {
                const bf16_t* p = reinterpret_cast<const bf16_t*>(o.a[j]) + k0;
                uint32_t e[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) e[i] = k0 + c + i < o.K ? (uint32_t)p[i] : 0u;
                r.a[j] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lin = j * 256 + tid, kr = lin >> 4, u = lin & 15;
            const int64_t at = (int64_t)(k0 + kr) * o.N + u * 8;
            uint32_t e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) e[i] = at + i < o.avail ? (uint32_t)o.B[at + i] : 0u;
            r.b[j] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
        }
    }
}

template <bool AF32>
__device__ __forceinline__ void any_write(const AnyRegs<AF32>& r, char* stage) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = j * 64 + (tid >> 2), c = tid & 3;
        char* p = stage + row * 64 + ((c ^ ((row >> 2) & 3)) * 16);
        if constexpr (AF32) {
            const uint4 u = r.a[2 * j], v = r.a[2 * j + 1];
            float f[8] = {__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w),
                          __uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
#pragma unroll
            for (int part = 0; part < 3; ++part) {
                uint4 o;
                o.x = bf16_part(f[0], f[1]); o.y = bf16_part(f[2], f[3]); o.z = bf16_part(f[4], f[5]); o.w = bf16_part(f[6], f[7]);
                *reinterpret_cast<uint4*>(p + (part == 0 ? 0 : kRest + (part - 1) * kATile)) = o;
            }
        } else {
            *reinterpret_cast<uint4*>(p) = r.a[j];
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int lin = j * 256 + tid, kr = lin >> 4, u = lin & 15;
        *reinterpret_cast<uint4*>(stage + kATile + kr * (ABN * 2) + b_lds_pos<ABN>(kr, u) * 16) = r.b[j];
    }
}

template <bool AF32>
__device__ __forceinline__ void any_compute(f32x16_t (&acc)[2][2], const char* stage, const FragAddr<ABM, ABN, 22>& f) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const bf16x8_t b[2] = {dma_read_b<ABM, ABN, 22, 0>(stage, f, kk), dma_read_b<ABM, ABN, 22, 1>(stage, f, kk)};
#pragma unroll
        for (int part = 0; part < (AF32 ? 3 : 1); ++part) {
            const char* at = stage + (part == 0 ? 0 : kRest + (part - 1) * kATile);
            const bf16x8_t a[2] = {dma_read_a<ABM, ABN, 22, 0>(at, f, kk), dma_read_a<ABM, ABN, 22, 1>(at, f, kk)};
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[ni], a[mi], acc[mi][ni], 0, 0, 0);
        }
    }
}

// acc = A B over k in [kbeg, kend); every wave leaves through the barrier behind the last read of LDS
template <bool AF32>
__device__ __forceinline__ void any_product(f32x16_t (&acc)[2][2], const void* A, int64_t lda, const bf16_t* B, int N, int K, int kbeg, int kend,
                                            int M, int m0, int n0, char* ring, const FragAddr<ABM, ABN, 22>& f) {
    constexpr int SB = any_stage_bytes<AF32>();
    const int tid = threadIdx.x;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 0.f;
    const int ns = (kend - kbeg + ABK - 1) / ABK;
    if (ns <= 0) return;
    AnyOperands o;
    o.B = B + n0; o.N = N; o.K = kend; o.avail = (int64_t)K * N - n0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        int m = m0 + j * 64 + (tid >> 2);
        m = m < M ? m : M - 1;                                     // rows past the end repeat the last one; never stored
        o.a[j] = reinterpret_cast<const char*>(A) + ((size_t)m * (size_t)lda + (size_t)((tid & 3) * 8)) * (AF32 ? 4 : 2);
    }
    AnyRegs<AF32> r0, r1;
    any_load<AF32>(r0, o, kbeg);
    if (ns > 1) any_load<AF32>(r1, o, kbeg + ABK);
    any_write<AF32>(r0, ring);
    if (ns > 2) any_load<AF32>(r0, o, kbeg + 2 * ABK);
    __syncthreads();
    for (int s = 0; s < ns; s += 2) {
        any_compute<AF32>(acc, ring, f);
        if (s + 1 < ns) any_write<AF32>(r1, ring + SB);
        if (s + 3 < ns) any_load<AF32>(r1, o, kbeg + (s + 3) * ABK);
        __syncthreads();
        if (s + 1 < ns) {
            any_compute<AF32>(acc, ring + SB, f);
            if (s + 2 < ns) any_write<AF32>(r0, ring);
            if (s + 4 < ns) any_load<AF32>(r0, o, kbeg + (s + 4) * ABK);
            __syncthreads();
        }
    }
}

// ---- sums of products in parts that are not finite ------------------------------------------------
// An infinite weight times a part that is zero is NaN, and so is every weight times an infinite value's rest.  Such elements are
// formed again in plain fp32.
// Nothing finite hides either (a sum that has met an infinity or NaN stays one, and so does SiLU(g) * u), so a tile pays a
// few comparisons while it is stored.
__device__ __forceinline__ bool not_finite(float v) { return !(__builtin_fabsf(v) < INFINITY); }
__device__ __forceinline__ bool not_finite_pair(uint32_t w) { return (w & 0x7f80u) == 0x7f80u || (w & 0x7f800000u) == 0x7f800000u; }
__device__ __forceinline__ float plain_dot(const void* A, int64_t lda, const void* B, int N, int m, int col, int k0, int k1) {
    const float* a = reinterpret_cast<const float*>(A) + (size_t)m * (size_t)lda;
    const bf16_t* w = reinterpret_cast<const bf16_t*>(B) + col;
    float s = 0.f;
#pragma unroll 1
    for (int k = k0; k < k1; ++k) s += a[k] * bf16_to_f32(w[(size_t)k * (size_t)N]);
    return s;
}
// The wave's 64 x 64 part of a stored tile at (r0, c0), a column per lane: whatever is not finite there, once more
template <int EPI>
__device__ __forceinline__ void mend_part(const AnyProb& P, int M, int r0, int c0, int sp, int k0, int k1) {
    const int col = c0 + (int)(threadIdx.x & 63), N = P.N;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // the part has been stored
#pragma unroll 1
    for (int m = r0; m < r0 + 64 && m < M; ++m) {
        if (col >= N) continue;
        if constexpr (EPI != ANY_OUT) {
            float* d = reinterpret_cast<float*>(P.C) + (size_t)sp * (size_t)P.split_stride + (size_t)m * (size_t)P.ldc + col;
            if (!not_finite(*d)) continue;
            float v = plain_dot(P.A, P.lda, P.B, N, m, col, k0, k1);
            if constexpr (EPI == ANY_GATEUP) {
                const float bg = P.bias ? bf16_to_f32(reinterpret_cast<const bf16_t*>(P.bias)[col]) : 0.f;
                const float bu = P.bias2 ? bf16_to_f32(reinterpret_cast<const bf16_t*>(P.bias2)[col]) : 0.f;
                v = silu_f32(v + bg) * (plain_dot(P.A2, P.lda2, P.B2, N, m, col, 0, P.K2) + bu);
            }
            *d = v;
        } else {
            bf16_t* const d = P.C ? reinterpret_cast<bf16_t*>(P.C) + (size_t)m * (size_t)P.ldc + col : nullptr;
            bf16_t* cd = nullptr;
            if (P.cache) {
                const int bi = m / P.T;
                const int64_t pp = (int64_t)P.pos[bi] + (m - bi * P.T);
                if (pp >= 0 && pp < P.S_max) cd = reinterpret_cast<bf16_t*>(P.cache) + ((size_t)bi * (size_t)P.S_max + (size_t)pp) * (size_t)N + col;
            }
            if ((!d && !cd) || !not_finite(bf16_to_f32(d ? *d : *cd))) continue;
            const float v = plain_dot(P.A, P.lda, P.B, N, m, col, k0, k1) + (P.bias ? bf16_to_f32(reinterpret_cast<const bf16_t*>(P.bias)[col]) : 0.f);
            if (d) *d = f32_to_bf16(v);
            if (cd) *cd = f32_to_bf16(v);
        }
    }
}

// nv of 8 consecutive bf16 columns, at any 2-byte alignment
__device__ __forceinline__ void store8(bf16_t* dst, const uint4& v, int nv) {
    if (nv >= 8) { __builtin_memcpy(dst, &v, 16); return; }
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (e < nv) dst[e] = (bf16_t)(w[e >> 1] >> (16 * (e & 1)));
}

template <bool AF32, int EPI>
__global__ void __launch_bounds__(256, 2) k_any_gemm(AnyArgs ga) {
    constexpr int SB = any_stage_bytes<AF32>();
    __shared__ uint4 lds[2 * SB / 16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    char* ring = reinterpret_cast<char*>(lds);
    char* patch = ring + wave * 4096;                              // (the products leave the ring through a barrier)
    // workgroups go to the 8 XCDs round-robin: give each XCD a contiguous run of tiles
    const int per = (ga.count + 7) >> 3;
    const int local = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (local >= ga.count) return;
    const int id = ga.first + local;
    int pi = 0;
#pragma unroll
    for (int i = 1; i < kMaxAny; ++i)
        if (i < ga.nprob && id >= ga.p[i].tile_begin) pi = i;
    const AnyProb& P = ga.p[pi];
    // chunk of K, then groups of 8 tile rows column by column
    int rem = id - P.tile_begin;
    const int tiles = ga.tiles_m * P.tiles_n;
    const int sp = rem / tiles; rem -= sp * tiles;
    const int gsz = 8 * P.tiles_n, mg = rem / gsz, r = rem - mg * gsz;
    const int rows = ga.tiles_m - mg * 8 < 8 ? ga.tiles_m - mg * 8 : 8;
    const int tn = r / rows, tm = mg * 8 + (r - tn * rows);
    const int m0 = tm * ABM, n0 = tn * ABN, M = ga.M, N = P.N;

    FragAddr<ABM, ABN, 22> f;
    frag_setup<ABM, ABN, 22>(f, wave);
    f32x16_t acc[2][2], acc2[EPI == ANY_GATEUP ? 2 : 1][EPI == ANY_GATEUP ? 2 : 1];
    const int kb = sp * P.kchunk, ke = kb + P.kchunk < P.K ? kb + P.kchunk : P.K;
    any_product<AF32>(acc, P.A, P.lda, reinterpret_cast<const bf16_t*>(P.B), N, P.K, kb, ke, M, m0, n0, ring, f);
    if constexpr (EPI == ANY_GATEUP)
        any_product<AF32>(acc2, P.A2, P.lda2, reinterpret_cast<const bf16_t*>(P.B2), N, P.K2, 0, P.K2, M, m0, n0, ring, f);

    // lane (li, lg) holds, for tile row 32 mi + li of its wave's quarter, columns 32 ni + 8 vg + 4 lg .. + 3; rows leave through
    // the wave's 4 KB patch (16-byte units swizzled by row) as 128 consecutive bytes
    const int wm = wave >> 1, wn = wave & 1, li = lane & 31, lg = lane >> 5;
    const int rrow = lane >> 3, runit = lane & 7;
    const bf16_t* bias = reinterpret_cast<const bf16_t*>(P.bias);
    const bf16_t* bias2 = reinterpret_cast<const bf16_t*>(P.bias2);
    bool again = false;                     // this lane has stored something that is not finite
    if constexpr (EPI != ANY_OUT) {
        float* const C = reinterpret_cast<float*>(P.C) + (size_t)sp * (size_t)P.split_stride;
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            float bg[4][4], bu[4][4];
            if constexpr (EPI == ANY_GATEUP) {
#pragma unroll
                for (int vg = 0; vg < 4; ++vg)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int col = n0 + wn * 64 + ni * 32 + 8 * vg + 4 * lg + e;
                        bg[vg][e] = bias && col < N ? bf16_to_f32(bias[col]) : 0.f;
                        bu[vg][e] = bias2 && col < N ? bf16_to_f32(bias2[col]) : 0.f;
                    }
            }
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
                for (int vg = 0; vg < 4; ++vg) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (EPI == ANY_GATEUP) v[e] = silu_f32(acc[mi][ni][4 * vg + e] + bg[vg][e]) * (acc2[mi][ni][4 * vg + e] + bu[vg][e]);
                        else v[e] = acc[mi][ni][4 * vg + e];
                    }
                    *reinterpret_cast<float4*>(patch + li * 128 + (((2 * vg + lg) ^ ((li >> 1) & 7)) * 16)) = make_float4(v[0], v[1], v[2], v[3]);
                }
                const int col = n0 + wn * 64 + ni * 32 + runit * 4;
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int row = it * 8 + rrow, m = m0 + wm * 64 + mi * 32 + row;
                    const float4 v = *reinterpret_cast<const float4*>(patch + row * 128 + ((runit ^ ((row >> 1) & 7)) * 16));
                    if (m < M && col < N) {
                        if constexpr (AF32) again = again || not_finite(v.x) || not_finite(v.y) || not_finite(v.z) || not_finite(v.w);
                        float* d = C + (size_t)m * (size_t)P.ldc + col;
                        if (col + 4 <= N) __builtin_memcpy(d, &v, 16);
                        else { d[0] = v.x; if (col + 1 < N) d[1] = v.y; if (col + 2 < N) d[2] = v.z; }
                    }
                }
            }
        }
    } else {
        bf16_t* const C = reinterpret_cast<bf16_t*>(P.C);
        bf16_t* const cache = reinterpret_cast<bf16_t*>(P.cache);
        const int col8 = n0 + wn * 64 + runit * 8;
        const int nv = N - col8;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            const int r0 = m0 + wm * 64 + mi * 32;
            int crow[4] = {-1, -1, -1, -1};
            if (cache) cache_rows(crow, P.pos, P.T, P.S_max, M, r0, rrow);
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int vg = 0; vg < 4; ++vg) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int col = n0 + wn * 64 + ni * 32 + 8 * vg + 4 * lg + e;
                        v[e] = acc[mi][ni][4 * vg + e] + (bias && col < N ? bf16_to_f32(bias[col]) : 0.f);
                    }
                    uint2 o; o.x = ppack2(v[0], v[1]); o.y = ppack2(v[2], v[3]);
                    *reinterpret_cast<uint2*>(patch + li * 128 + (((ni * 4 + vg) ^ ((li >> 1) & 7)) * 16) + lg * 8) = o;
                }
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int row = it * 8 + rrow, m = r0 + row;
                const uint4 v = *reinterpret_cast<const uint4*>(patch + row * 128 + ((runit ^ ((row >> 1) & 7)) * 16));
                if constexpr (AF32) again = again || not_finite_pair(v.x) || not_finite_pair(v.y) || not_finite_pair(v.z) || not_finite_pair(v.w);
                if (nv > 0 && m < M && C) store8(C + (size_t)m * (size_t)P.ldc + col8, v, nv);
                if (nv > 0 && crow[it] >= 0) store8(cache + (size_t)crow[it] * (size_t)N + col8, v, nv);
            }
        }
    }
    if constexpr (AF32) {
        if (__builtin_amdgcn_ballot_w64(again) != 0ull) mend_part<EPI>(P, M, m0 + wm * 64, n0 + wn * 64, sp, kb, ke);
    }
}

// dst[i] = sum over `splits` of part[i + sp * stride], in chunk order
__global__ void __launch_bounds__(256) k_any_reduce(const float* __restrict__ part, float* __restrict__ dst, int64_t n, int splits, int64_t stride) {
    for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i < n; i += (int64_t)gridDim.x * 1024) {
        float4 a = *reinterpret_cast<const float4*>(part + i);            // (the partial areas are padded to whole float4s)
        for (int sp = 1; sp < splits; ++sp) {
            const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)sp * stride + i);
            a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
        }
        if (i + 4 <= n) *reinterpret_cast<float4*>(dst + i) = a;
        else { dst[i] = a.x; if (i + 1 < n) dst[i + 1] = a.y; if (i + 2 < n) dst[i + 2] = a.z; }
    }
}

int any_launch_bf16(AnyArgs& a, bool a_f32, int epi, hipStream_t s) {
    a.tiles_m = (a.M + ABM - 1) / ABM;
    int64_t total = 0;
    for (int i = 0; i < a.nprob; ++i) {
        AnyProb& p = a.p[i];
        p.tiles_n = (p.N + ABN - 1) / ABN; p.tile_begin = (int)total;
        if (p.kchunk <= 0) p.kchunk = p.K > 0 ? p.K : 1;
        total += (int64_t)a.tiles_m * p.tiles_n * p.splits;
    }
    if (total <= 0) return LR_OK;
    if (total >= (1ll << 31)) { set_error("too many output tiles"); return LR_ERR_UNSUPPORTED; }
    for (int64_t first = 0; first < total; first += kAnyLaunchTiles) {
        a.first = (int)first;
        a.count = (int)(total - first < kAnyLaunchTiles ? total - first : kAnyLaunchTiles);
        const dim3 grid((unsigned)((a.count + 7) / 8 * 8)), block(256);
        if (epi == ANY_T) {
            if (a_f32) hipLaunchKernelGGL((k_any_gemm<true, ANY_T>), grid, block, 0, s, a);
            else       hipLaunchKernelGGL((k_any_gemm<false, ANY_T>), grid, block, 0, s, a);
        } else if (epi == ANY_GATEUP) hipLaunchKernelGGL((k_any_gemm<true, ANY_GATEUP>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_any_gemm<true, ANY_OUT>), grid, block, 0, s, a);
        const int st = launch_status("product of any sizes");
        if (st != LR_OK) return st;
    }
    return LR_OK;
}

int any_reduce(const float* part, float* dst, int64_t n, int splits, int64_t stride, hipStream_t s) {
    int64_t blocks = (n / 4 + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_any_reduce, dim3((unsigned)blocks), dim3(256), 0, s, part, dst, n, splits, stride);
    return launch_status("sum of K chunks");
}

}  // namespace lr
