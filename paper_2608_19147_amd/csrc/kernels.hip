// gfx950 kernels of the stage forward.
//
// gemv_kernel  : W4A16 matrix-vector product for up to 8 activation rows.  One
//                wave lane owns one weight row of a 64-row tile and streams
//                16-byte chunks (32 INT4 codes) with non-temporal loads; the
//                activation slice sits in LDS as fp16 pairs and is broadcast to
//                all lanes; codes become fp16 with the 0x6400 mask-and-or trick
//                and are consumed by v_dot2_f32_f16 (fp32 accumulation); the
//                group scale multiplies each chunk's partial dot product, so the
//                dequantized weight is exact.  Prologue: RMSNorm of the input
//                row.  Epilogue: plain store, residual add, or SwiGLU.  K is split
//                over workgroups; the last workgroup of a tile (atomic ticket)
//                sums the partials in a fixed order, so results are deterministic.
// attn_kernel  : split-KV decode/verify attention.  Grid = (slot, kv head,
//                split); 16 lanes read one 256-byte cache row, 16 rows per step
//                per workgroup.  Rows j < P are read through the beam table;
//                rows j >= P are this forward's new k/v, rotated and rounded here
//                and written to the cache by their owner.  Mask and causality
//                decide visibility inside an online softmax (exp2 domain);
//                attn_merge_kernel then combines the split partials.
#include "device.h"

#include <climits>

namespace stg {

__device__ __forceinline__ int dest_row(int r, int row_off, int row_map) {
    if (row_map == 0) return row_off + r;
    return 64 * (r >> 5) + (r & 31) + (row_map == 2 ? 32 : 0);   // gate | up interleave
}

// ------------------------------------------------------------------ repack

__global__ void repack_codes_kernel(const uint8_t* __restrict__ q, int n, int k, uint8_t* __restrict__ w_out,
                                    int nchunk, int row_off, int row_map) {
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= (size_t)n * nchunk) return;
    const int r = (int)(idx / nchunk), c = (int)(idx % nchunk);
    const int kb = (k + 1) / 2;
    const int dr = dest_row(r, row_off, row_map);
    const int t = dr >> 6, lane = dr & 63;
    u32x4 o;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        uint32_t wd = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int kk = c * 32 + d * 8 + e;
            uint32_t nib = 8;
            if (kk < k) {
                const uint8_t byte = q[(size_t)r * kb + (kk >> 1)];
                nib = (kk & 1) ? (byte >> 4) : (byte & 15);
            }
            const int sh = (e & 1) ? (16 + 4 * (e >> 1)) : 4 * (e >> 1);
            wd |= nib << sh;
        }
        o[d] = wd;
    }
    *(u32x4*)(w_out + (((size_t)t * nchunk + c) * 64 + lane) * 16) = o;
}

__global__ void repack_scales_kernel(const uint16_t* __restrict__ s, int n, int ng, uint16_t* __restrict__ s_out,
                                     int ngroups, int row_off, int row_map) {
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= (size_t)n * ng) return;
    const int r = (int)(idx / ng), g = (int)(idx % ng);
    const int dr = dest_row(r, row_off, row_map);
    const int t = dr >> 6, lane = dr & 63;
    s_out[((size_t)t * ngroups + g) * 64 + lane] = s[idx];
}

hipError_t launch_repack(const uint8_t* q, const uint16_t* s, int n, int k, int g, uint8_t* w_out, uint16_t* s_out,
                         int ntiles, int nchunk, int ngroups, int row_off, int row_map, hipStream_t st) {
    (void)ntiles;
    const size_t nc = (size_t)n * nchunk;
    repack_codes_kernel<<<dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st>>>(q, n, k, w_out, nchunk, row_off, row_map);
    const int ng = (k + g - 1) / g;
    const size_t ns = (size_t)n * ng;
    repack_scales_kernel<<<dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, st>>>(s, n, ng, s_out, ngroups, row_off, row_map);
    return hipGetLastError();
}

// ------------------------------------------------------------------ debug dequant

__global__ void dequant_kernel(PackedMat m, int row_off, int row_map, int n_rows, float* __restrict__ out) {
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= (size_t)n_rows * m.nchunk) return;
    const int r = (int)(idx / m.nchunk), c = (int)(idx % m.nchunk);
    const int dr = dest_row(r, row_off, row_map);
    const int t = dr >> 6, lane = dr & 63;
    const u32x4 w = *(const u32x4*)(m.w + (((size_t)t * m.nchunk + c) * 64 + lane) * 16);
    half2_t h[16];
    unpack_chunk(w, h);
    const float sc = f16_to_f32(m.s[((size_t)t * m.ngroups + c / m.gchunks) * 64 + lane]);
#pragma unroll
    for (int p = 0; p < 16; ++p) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int kk = c * 32 + 2 * p + e;
            if (kk < m.k) out[(size_t)r * m.k + kk] = (float)h[p][e] * sc;
        }
    }
}

hipError_t launch_dequant(const PackedMat& m, int row_off, int row_map, int n_rows, float* out, hipStream_t st) {
    const size_t nc = (size_t)n_rows * m.nchunk;
    dequant_kernel<<<dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st>>>(m, row_off, row_map, n_rows, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ GEMV

// Inverse RMS of M input rows of length K, fp32, deterministic order.
template <int MT>
__device__ __forceinline__ void rms_fullrow(const GemvArgs& a, int K, float* rs_s, float* bsum) {
    const int tid = threadIdx.x;
    for (int m = 0; m < a.M; ++m) {
        float ss = 0.f;
        for (int k8 = tid; k8 < K / 8; k8 += 256) {
            float v[8];
            const size_t base = (size_t)m * a.in_ld + 8 * k8;
            if (a.in_dt == DT_F32) {
                const float4 p = *(const float4*)((const float*)a.in + base);
                const float4 q = *(const float4*)((const float*)a.in + base + 4);
                v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = p.w; v[4] = q.x; v[5] = q.y; v[6] = q.z; v[7] = q.w;
            } else {
                const u32x4 h = *(const u32x4*)((const uint16_t*)a.in + base);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t w = h[e >> 1];
                    v[e] = half_bits_to_f32((uint16_t)((e & 1) ? (w >> 16) : (w & 0xFFFFu)), a.in_dt);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
        }
        ss = block_sum256(ss, bsum);
        if (tid == 0) rs_s[m] = rsqrtf(ss / (float)K + a.eps);
    }
}

template <int MT, int CPW>
__global__ __launch_bounds__(256) void gemv_kernel(GemvArgs a) {
    constexpr int CPS = 4 * CPW;                 // chunks per workgroup
    constexpr int KLEN = CPS * 32;               // k values per workgroup
    constexpr int NI = (MT * KLEN / 8 + 255) / 256;
    constexpr int NV = (MT * 64 + 255) / 256;
    __shared__ __attribute__((aligned(16))) uint32_t xs[MT][KLEN / 2];
    __shared__ float red[4][MT][64];
    __shared__ float rs_s[MT];
    __shared__ float bsum[256];
    __shared__ int last_s;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = blockIdx.x, s = blockIdx.y;
    const PackedMat W = a.W;
    const int M = a.M;
    const int K = W.k;
    const int c0 = s * CPS;
    const int k0 = c0 * 32;

    // ---- weights of this wave: issue every load first (activation-independent)
    const int cw0 = c0 + wave * CPW;
    const u32x4* wbase = (const u32x4*)W.w + ((size_t)t * W.nchunk + cw0) * 64 + lane;
    u32x4 wv[CPW];
    uint16_t sraw[CPW];
#pragma unroll
    for (int u = 0; u < CPW; ++u) wv[u] = __builtin_nontemporal_load(wbase + (size_t)u * 64);
    const uint16_t* sbase = W.s + (size_t)t * W.ngroups * 64 + lane;
#pragma unroll
    for (int u = 0; u < CPW; ++u) sraw[u] = sbase[(size_t)((cw0 + u) / W.gchunks) * 64];

    // ---- prologue: inverse RMS of each input row
    if (a.rms == RMS_FULLROW) {
        rms_fullrow<MT>(a, K, rs_s, bsum);
    } else if (a.rms == RMS_PARTIALS) {
        // wave w reduces rows w, w + 4, ...: lane l adds tiles l, l + 64, ... in order,
        // then lane 0 receives a fixed-order butterfly sum
        for (int m = wave; m < M; m += 4) {
            float ss = 0.f;
            for (int tt = lane; tt < a.ssq_tiles; tt += 64) ss += a.ssq_in[(size_t)m * a.ssq_tiles + tt];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
            if (lane == 0) rs_s[m] = rsqrtf(ss / (float)K + a.eps);
        }
    }
    __syncthreads();

    // ---- stage the activation slice [k0, k0 + KLEN) as fp16 pairs, 8 k per item
    {
        float v[NI][8];
        float gm[NI][8];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int it = tid + 256 * i;
            const int m = it / (KLEN / 8);
            const int kk = k0 + 8 * (it % (KLEN / 8));
            const bool ok = (it < M * (KLEN / 8)) && (kk < K);
            const size_t base = ok ? (size_t)m * a.in_ld + kk : 0;
            if (a.in_dt == DT_F32) {
                const float4 p = *(const float4*)((const float*)a.in + base);
                const float4 q = *(const float4*)((const float*)a.in + base + 4);
                v[i][0] = p.x; v[i][1] = p.y; v[i][2] = p.z; v[i][3] = p.w;
                v[i][4] = q.x; v[i][5] = q.y; v[i][6] = q.z; v[i][7] = q.w;
            } else {
                const u32x4 h = *(const u32x4*)((const uint16_t*)a.in + base);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t w = h[e >> 1];
                    v[i][e] = half_bits_to_f32((uint16_t)((e & 1) ? (w >> 16) : (w & 0xFFFFu)), a.in_dt);
                }
            }
            if (a.rms != RMS_NONE) {
                const u32x4 g = *(const u32x4*)(a.gamma + (ok ? kk : 0));
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t w = g[e >> 1];
                    gm[i][e] = half_bits_to_f32((uint16_t)((e & 1) ? (w >> 16) : (w & 0xFFFFu)), a.gamma_dt);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (!ok) v[i][e] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int it = tid + 256 * i;
            if (it < M * (KLEN / 8)) {
                const int m = it / (KLEN / 8);
                const int p0 = 4 * (it % (KLEN / 8));
                if (a.rms != RMS_NONE) {
                    const float rs = rs_s[m];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[i][e] = (v[i][e] * rs) * gm[i][e];
                }
                u32x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = pack_f16x2(v[i][2 * q], v[i][2 * q + 1]);
                *(u32x4*)&xs[m][p0] = o;
            }
        }
    }
    __syncthreads();

    // ---- dot products (codes exact in fp16, fp32 accumulation, scale per chunk)
    float acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = 0.f;
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
        half2_t wq[16];
        unpack_chunk(wv[u], wq);
        const float sc = f16_to_f32(sraw[u]);
        const int pc = (wave * CPW + u) * 16;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            if (m < M) {
                const u32x4* xv = (const u32x4*)&xs[m][pc];
                float d = 0.f;
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const u32x4 x4 = xv[q4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        // copy the element out first: a bit_cast of a vector-element
                        // lvalue reads element 0 of the vector
                        const uint32_t xe = x4[e];
                        d = __builtin_amdgcn_fdot2(wq[4 * q4 + e], __builtin_bit_cast(half2_t, xe), d, false);
                    }
                }
                acc[m] += sc * d;
            }
        }
    }

    // ---- reduce the four waves (fixed order)
#pragma unroll
    for (int m = 0; m < MT; ++m) red[wave][m][lane] = acc[m];
    __syncthreads();
    float vals[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int idx = tid + 256 * q;
        vals[q] = 0.f;
        if (idx < M * 64) {
            const int m = idx >> 6, r = idx & 63;
            vals[q] = ((red[0][m][r] + red[1][m][r]) + red[2][m][r]) + red[3][m][r];
        }
    }

    // ---- split-K: the last workgroup of the tile sums every split in split order
    if (a.ksplit > 1) {
        const int ldp = W.ntiles * 64;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (idx < M * 64)
                store_coherent(&a.partial[((size_t)s * M + (idx >> 6)) * ldp + t * 64 + (idx & 63)], vals[q]);
        }
        if (!last_arrival(&a.counters[t], (unsigned)a.ksplit, &last_s)) return;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (idx < M * 64) {
                const float* pp = &a.partial[(size_t)(idx >> 6) * ldp + t * 64 + (idx & 63)];
                const size_t stride = (size_t)M * ldp;
                float v = 0.f;
                int ss = 0;
                for (; ss + 8 <= a.ksplit; ss += 8) {
                    float b8[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) b8[e] = load_coherent(pp + (ss + e) * stride);
#pragma unroll
                    for (int e = 0; e < 8; ++e) v += b8[e];
                }
                for (; ss < a.ksplit; ++ss) v += load_coherent(pp + ss * stride);
                vals[q] = v;
            }
        }
    }

    // ---- epilogue
    if (a.epi == EPI_STORE) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (idx < M * 64) {
                const int m = idx >> 6, n = t * 64 + (idx & 63);
                if (n < W.n) a.out[(size_t)m * a.out_ld + n] = vals[q];
            }
        }
    } else if (a.epi == EPI_RESID) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (idx < M * 64) {
                const int m = idx >> 6, r = idx & 63;
                const int n = t * 64 + r;
                float xn = 0.f;
                if (n < W.n) {
                    xn = load_val(a.resid, a.resid_dt, (size_t)m * a.resid_ld + n) + vals[q];
                    a.out[(size_t)m * a.out_ld + n] = xn;
                    if (a.out_act) ((uint16_t*)a.out_act)[(size_t)m * a.out_act_ld + n] = to_half_bits(xn, a.out_act_dt);
                }
                red[0][m][r] = xn * xn;
            }
        }
        __syncthreads();
        if (a.ssq_out && tid < M) {
            float ss = 0.f;
            for (int r = 0; r < 64; ++r) ss += red[0][tid][r];
            a.ssq_out[(size_t)tid * W.ntiles + t] = ss;
        }
    } else {  // EPI_SWIGLU: rows 0..31 of the tile are gate rows, 32..63 the matching up rows
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (idx < M * 64) red[0][idx >> 6][idx & 63] = vals[q];
        }
        __syncthreads();
        for (int idx = tid; idx < M * 32; idx += 256) {
            const int m = idx >> 5, r = idx & 31;
            const int f = t * 32 + r;
            if (f < a.n_valid) {
                const float gt = red[0][m][r], up = red[0][m][r + 32];
                a.out[(size_t)m * a.out_ld + f] = (gt / (1.0f + expf(-gt))) * up;
            }
        }
    }
}

template <int MT>
hipError_t launch_gemv_m(const GemvArgs& a, int cpw, hipStream_t st) {
    const dim3 grid(a.W.ntiles, a.ksplit), block(256);
    switch (cpw) {
        case 1: gemv_kernel<MT, 1><<<grid, block, 0, st>>>(a); break;
        case 2: gemv_kernel<MT, 2><<<grid, block, 0, st>>>(a); break;
        case 4: gemv_kernel<MT, 4><<<grid, block, 0, st>>>(a); break;
        case 8: gemv_kernel<MT, 8><<<grid, block, 0, st>>>(a); break;
        case 16: gemv_kernel<MT, 16><<<grid, block, 0, st>>>(a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gemv(const GemvArgs& a, hipStream_t st) {
    if (a.cps % 4) return hipErrorInvalidValue;
    const int cpw = a.cps / 4;
    switch (a.M) {
        case 1: return launch_gemv_m<1>(a, cpw, st);
        case 2: return launch_gemv_m<2>(a, cpw, st);
        case 3: return launch_gemv_m<3>(a, cpw, st);
        case 4: return launch_gemv_m<4>(a, cpw, st);
        case 5: return launch_gemv_m<5>(a, cpw, st);
        case 6: return launch_gemv_m<6>(a, cpw, st);
        case 7: return launch_gemv_m<7>(a, cpw, st);
        case 8: return launch_gemv_m<8>(a, cpw, st);
        default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------ GEMM (matrix cores)

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// (x & m) | c, written as plain arithmetic (one v_and_or_b32).  Its results feed
// matrix-core operands, so it must stay visible to the compiler: the wait states
// required between a vector write and a matrix-core read of the same register
// are inserted only for instructions the compiler itself emits.
__device__ __forceinline__ uint32_t and_or_u32(uint32_t m, uint32_t x, uint32_t c) { return (x & m) | c; }

// ------------------------------------------------------------------ prepared-operand products
//
// For 2..64 rows the input of every product is written once by the kernel that
// produces it, in the form the matrix cores take: fp16 h with the values at
// positions 2, 3, 6, 7 of every 8 k divided by 16 (they meet codes decoded as
// 1024 + 16u), plus per 32 k the correction 1032 * sum(h at 0, 1, 4, 5) +
// 72 * sum(h at 2, 3, 6, 7) that removes the decode offsets.  An RMSNorm input
// is prepared as h = x * gamma * c with c the row's previous normalization
// scale; the product multiplies its results by rs / c once rs is known
// (RMSNorm(x) W^T = rs ((x * gamma) W^T)).

__device__ __forceinline__ uint16_t bp_code(float h16, int k) { return f32_to_f16((k & 2) ? h16 * 0.0625f : h16); }
__device__ __forceinline__ float bp_corr(float h16, int k) { return ((k & 2) ? 72.0f : 1032.0f) * h16; }

// Sum over the 64 lanes of a wave, identical in every lane.
__device__ __forceinline__ float wave_sum_all(float v) {
    v = sum16(v);
    uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    u = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// Largest value / smallest integer over the wave, identical in every lane.
// (lane exchanges within the vector unit; through LDS each of the six took a round trip).
__device__ __forceinline__ float wave_max_all(float v) {
    v = fmaxf(v, dpp_f<0xB1>(v));
    v = fmaxf(v, dpp_f<0x4E>(v));
    v = fmaxf(v, dpp_f<0x141>(v));
    v = fmaxf(v, dpp_f<0x140>(v));
    uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = __float_as_uint(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
    const auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false); }
__device__ __forceinline__ int wave_min_all(int v) {
    v = min(v, dpp_i<0xB1>(v));
    v = min(v, dpp_i<0x4E>(v));
    v = min(v, dpp_i<0x141>(v));
    v = min(v, dpp_i<0x140>(v));
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min((int)r[0], (int)r[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return min((int)q[0], (int)q[1]);
}

// Sum over aligned groups of 32 lanes, identical in every lane of the group.
__device__ __forceinline__ float sum32_lanes(float v) {
    v += dpp_f<0xB1>(v);              // lane ^ 1
    v += dpp_f<0x4E>(v);              // lane ^ 2
    v += dpp_f<0x124>(v);             // row_ror:4
    v += dpp_f<0x128>(v);             // row_ror:8: the 16-lane row
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Prepared operands are stored in the order the products read them: per group
// of 128 k, per column block cb (16 rows) and product i (k = 32 lg + 8 i + e
// within the group, lg = 0..3), the 64 lanes' 16 bytes (lane 16 lg + row mod
// 16) one after the other, so every operand load is one contiguous kilobyte.
// Corrections are [group][row][4 chunks of 32 k].
__device__ __forceinline__ size_t bp_index(int m, int k) {
    return ((((size_t)(k >> 7) * 16 + (m >> 4) * 4 + ((k >> 3) & 3)) * 64 + ((k >> 5) & 3) * 16 + (m & 15)) << 3) + (k & 7);
}
__device__ __forceinline__ size_t bc_index(int m, int k) { return ((size_t)(k >> 7) * 64 + m) * 4 + ((k >> 5) & 3); }

// One element of a prepared row: lanes 32 c .. 32 c + 31 of a wave hold k = 32 c' + (lane mod 32)
// of one row (valid = k < K); writes the code and, from lane 0 of the 32, the chunk's correction.
__device__ __forceinline__ void bp_put(uint16_t* bp, float* bc, int kp, int m, int k, float h, bool valid) {
    (void)kp;
    const float h16 = valid ? f16_to_f32(f32_to_f16(h)) : 0.f;
    const float cs = sum32_lanes(valid ? bp_corr(h16, k) : 0.f);
    if (valid) bp[bp_index(m, k)] = bp_code(h16, k);
    if (valid && (k & 31) == 0) bc[bc_index(m, k)] = cs;
}

// First q|k|v input of a forward: RMSNorm of the stage input row m, fully
// normalized (c = rs; the product's factor is 1); rs also goes to rs_out for
// the residual product that prepares the next input.  blockIdx.y takes one
// slice of BPREP_SLICE k: every slice adds the whole row's squares in the same
// order (so all get the same rs) and prepares only its own slice.
constexpr int BPREP_SLICE = 1024;
__global__ __launch_bounds__(256) void bprep_kernel(const void* in, int in_dt, int in_ld, const uint16_t* gamma,
                                                    int gamma_dt, int K, float eps, uint16_t* bp, float* bc, int kp,
                                                    float* rs_out) {
    constexpr int NPT = 32;                              // values per thread held in registers: K <= 8192
    constexpr int SPT = BPREP_SLICE / 256;               // slice values per thread
    __shared__ float red[4];
    const int m = blockIdx.x, tid = threadIdx.x, k0 = BPREP_SLICE * blockIdx.y;
    float v[NPT], xs[SPT], gs[SPT];
    size_t off[NPT], offs[SPT];                          // every load issued before any is used (clamped, then dropped)
#pragma unroll
    for (int i = 0; i < NPT; ++i) off[i] = (size_t)m * in_ld + min(tid + 256 * i, K - 1);
#pragma unroll
    for (int i = 0; i < SPT; ++i) offs[i] = (size_t)m * in_ld + min(k0 + tid + 256 * i, K - 1);
    load_vals(in, in_dt, off, v);
    load_vals(in, in_dt, offs, xs);
#pragma unroll
    for (int i = 0; i < SPT; ++i) gs[i] = half_bits_to_f32(gamma[min(k0 + tid + 256 * i, K - 1)], gamma_dt);
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NPT; ++i) ss += tid + 256 * i < K ? v[i] * v[i] : 0.f;
    ss = wave_sum_all(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float rs = rsqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)K + eps);
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
        const int k = k0 + tid + 256 * i;
        if (k0 + 256 * i < K) bp_put(bp, bc, kp, m, k, xs[i] * rs * gs[i], k < K);   // whole 32-lane groups
    }
    if (blockIdx.y == 0 && tid == 0) rs_out[m] = rs;
}

// Inputs of the row factors: the first 32 of this thread's quarter of row m's
// sums of squares (4 threads per row; loads clamped, then dropped past cnt),
// issued early so that they fly with the first group's loads.
struct RowFactorLoads {
    float v[32];
    float cb;
    int cnt;
    const float* src;
};
__device__ __forceinline__ void row_factor_loads(const GemvArgs& a, RowFactorLoads& r) {
    const int tid = threadIdx.x, m = tid >> 2, part = tid & 3;
    r.cb = 1.f;
    r.cnt = 0;
    r.src = a.ssq_in;
    if (a.norm == 1 && m < a.M) {
        r.cb = a.cb_in[m];
        const int per = (a.ssq_tiles + 3) / 4;
        r.src = a.ssq_in + (size_t)m * a.ssq_tiles + part * per;
        r.cnt = max(0, min(per, a.ssq_tiles - part * per));
        if (r.cnt > 0) {
#pragma unroll
            for (int e = 0; e < 32; ++e) r.v[e] = r.src[min(e, r.cnt - 1)];
        }
    }
}

// Factor of every row m < 64 of a product's results into fs (1 unless the
// input is a deferred RMSNorm: then rs / c, rs from the row's sums of squares,
// added by 4 threads per row in index order and combined in a fixed order);
// with write_rs, rs also goes to a.rs_out.  No barrier: fs is read after the
// workgroup's next one.
__device__ __forceinline__ void row_factors_finish(const GemvArgs& a, int K, bool write_rs, const RowFactorLoads& r,
                                                   float* fs) {
    const int tid = threadIdx.x, m = tid >> 2, part = tid & 3;
    float ss = 0.f;
    if (a.norm == 1 && m < a.M) {
#pragma unroll
        for (int e = 0; e < 32; ++e) ss += (e < r.cnt) ? r.v[e] : 0.f;
        for (int tt = 32; tt < r.cnt; tt += 32) {             // more than 128 partials per row
            float v[32];
#pragma unroll
            for (int e = 0; e < 32; ++e) v[e] = r.src[min(tt + e, r.cnt - 1)];
#pragma unroll
            for (int e = 0; e < 32; ++e) ss += (tt + e < r.cnt) ? v[e] : 0.f;
        }
    }
    ss += dpp_f<0xB1>(ss);                                    // lane ^ 1
    ss += dpp_f<0x4E>(ss);                                    // lane ^ 2: the row's 4 parts
    if (part == 0 && m < 64) {                                // (a 512-thread workgroup's upper half has no row)
        float f = 1.f;
        if (a.norm == 1 && m < a.M) {
            const float rs = rsqrtf(ss / (float)K + a.eps);
            f = rs / r.cb;
            if (write_rs && a.rs_out) a.rs_out[m] = rs;
        }
        fs[m] = f;
    }
}

// A bounds-checked buffer over `bytes` at p: a load whose lane offset lies past
// the end returns zero.  The uniform offset of buf_load16 is not checked: it only
// takes places that are in range.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
template <int AUX = 0>                                        // 2: non-temporal
__device__ __forceinline__ u32x4 buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, AUX));
}

// Product of the prepared input with one matrix: a workgroup's 4 waves take
// one 64-row tile and 4 consecutive ranges of a.kg groups of 128 k; blockIdx.y
// is the split of K (fixed per matrix, so results do not depend on M).  A lane
// loads 16 bytes of codes per row block and group (chunk 4 gi + lane / 16 of row
// 16 rt + lane mod 16): dword i of it, decoded, is an operand of the group's
// i-th product, whose k are 32 (4 gi + lane / 16) + 8 i + e; the other operand
// is read from the prepared rows at the same k.  The prepared rows are the
// products' rows and the weight rows their columns, so a lane's results belong
// to one weight row (one scale) and four input rows, whose corrections are the
// products' starting value: one fp32 product of the 16 rows' four corrections
// with -1.  That leaves one multiply-add per result and group.
// Z = 2: 33..64 rows, as two workgroups of 32 rows per tile that run one after
// the other on one XCD (the second finds the codes in its L2).
// PT = 2 (17 or more rows of a product that is neither split over K nor adds to
// a residual): eight waves take two tiles; the two waves of a K range fetch half
// of its prepared rows each and share them through LDS.  With every wave fetching
// its own, the caches delivered about 9.5 TB/s and bound the product: the LM
// head (20 rows, 8 KB of rows per 4 KB of codes) streamed its codes at 3.1 TB/s,
// at 16 rows (4 KB) 4.3.
template <int NCB, int Z, int PT>
__global__ __launch_bounds__(256 * PT, 2) void gemm_bp_kernel(GemvArgs a) {
    constexpr int MP = 16 * NCB;
    constexpr int NV = MP * 64 / 256;
    // the shared rows [buffer][K range][fragment][lane] (PT = 2) and, after the
    // products, the waves' sums [tile][wave][row][65].  PT = 2 takes more than half
    // of a CU's 160 KB, though its registers already admit one workgroup per CU: LM
    // head of 20 rows 87.5 us at 81 KB, 88.6 at the 65 KB it needs; 64 rows 4.30 and
    // 4.31 ms.
    constexpr int REDB = PT * 4 * MP * 65 * 4, RAWB = PT == 2 ? 81 * 1024 : REDB;
    static_assert(RAWB >= REDB && (PT == 1 || RAWB >= 2 * 4 * 4 * NCB * 1024), "LDS of the rows and the sums");
    __shared__ __attribute__((aligned(16))) uint8_t raw[RAWB];
    __shared__ float fs[64];
    constexpr bool PRE = NCB >= 2 && PT == 1;
    __shared__ float sres[PRE ? MP : 1][64], sgam[PRE ? 64 : 1], srs[PRE ? MP : 1];   // residual-epilogue inputs read at the start
    __shared__ int last_s;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = wave & 3;   // uniform: scalar loop control
    const int tl = wave >> 2, tid = threadIdx.x & 255, lane = tid & 63;   // tile of the workgroup, thread of the tile
    const int l16 = lane & 15, lg = lane >> 4;
    const int wg = Z == 1 ? (int)blockIdx.x : (int)((blockIdx.x >> 4) * 8 + (blockIdx.x & 7)), s = blockIdx.y;
    const int m0 = Z == 1 ? 0 : 32 * ((blockIdx.x >> 3) & 1);   // first row
    const PackedMat W = a.W;
    if (Z > 1 && PT * wg >= W.ntiles) return;                   // whole workgroup
    const bool has = PT * wg + tl < W.ntiles;
    const int t = has ? PT * wg + tl : W.ntiles - 1;            // an odd matrix's missing tile repeats the last; its results are dropped
    float (*red)[MP][65] = (float (*)[MP][65])(raw + (size_t)tl * 4 * MP * 65 * 4);
    const int M = a.M, K = W.k;
    // groups of K itself: the matrix may be padded by more, the prepared rows are not
    const int g0 = (4 * s + w) * a.kg, g1 = min((K + 127) / 128, g0 + a.kg);
    uint32_t magic = 0x64006400u;
    asm volatile("" : "+v"(magic));
    const __amdgpu_buffer_rsrc_t rw = buf_rsrc(W.w + (size_t)t * W.nchunk * 1024, (uint32_t)W.nchunk * 1024);
    const __amdgpu_buffer_rsrc_t rsc = buf_rsrc(W.s + (size_t)t * W.ngroups * 64, (uint32_t)W.ngroups * 128);
    const __amdgpu_buffer_rsrc_t rb = buf_rsrc(a.bp_in, (uint32_t)a.kp * 128);
    const __amdgpu_buffer_rsrc_t rc = buf_rsrc(a.bc_in, (uint32_t)a.kp * 8);
    const uint32_t wo = 16u * (64 * lg + l16), so = 2u * l16, bo = 16u * lane + 256u * m0, co = 16u * (m0 + l16) + 4u * lg;

    auto ldw = [&](int gi, u32x4 (&wv)[4], uint16_t (&sv)[4]) {
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) {
            wv[rt] = buf_load16<Z == 1 ? 2 /* nt */ : 0>(rw, wo, 4096 * gi + 256 * rt);
            sv[rt] = __builtin_amdgcn_raw_buffer_load_b16(rsc, so, 128 * gi + 32 * rt, 0);
        }
    };
    auto ldc = [&](int gi, float (&cv)[NCB]) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            cv[cb] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc, co, 1024 * gi + 256 * cb, 0));
    };
    // prepared operand and corrections (row l16, chunk lg) of one group as stored;
    // entries at k >= K (past the end of a ragged last group) are dropped when the
    // group computes, so nothing waits for these loads before then
    auto ldb = [&](int gi, u32x4 (&bv)[NCB][4], float (&cv)[NCB]) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) bv[cb][i] = buf_load16<0>(rb, bo, 16384 * gi + 4096 * cb + 1024 * i);
        }
        ldc(gi, cv);
    };

    f32x4_t acc[4][NCB];
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[rt][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // Two register sets, each the codes, scales, prepared operand and corrections
    // of one group: while one group computes, the next one's loads are in flight.
    // A group's loads are issued together (loads retire from the wait counter in
    // issue order) and unconditionally (the group index is clamped to the wave's
    // last; a repeated group is simply not computed), and nothing reads them
    // before the group computes, so no branch or select sits between a load and
    // its use and the compiler waits for exactly the loads each product needs.
    u32x4 wr[2][4], br[2][NCB][4];
    uint16_t sr[2][4];
    float cr[2][NCB];
    // PT = 2: this wave's half of the rows of its K range
    u32x4 rh[2 * NCB];
    u32x4 (*sb)[4][4 * NCB][64] = (u32x4 (*)[4][4 * NCB][64])raw;
    auto ldh = [&](int gi) {
#pragma unroll
        for (int u = 0; u < 2 * NCB; ++u) {
            const int f = 2 * NCB * tl + u;
            rh[u] = buf_load16<0>(rb, bo, 16384 * gi + 1024 * f);
        }
    };
    auto puth = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 2 * NCB; ++u) sb[buf][w][2 * NCB * tl + u][lane] = rh[u];
    };
    auto compute = [&](int gi, const u32x4 (&wv)[4], const uint16_t (&sv)[4], u32x4 (&bv)[NCB][4], float (&cv)[NCB]) {
        const int kb = 128 * gi;
        if (kb + 128 > K) {                              // a ragged last group (uniform)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {            // in place: the set is reloaded after this group
                    const bool in = kb + 32 * lg + 8 * i < K;
#pragma unroll
                    for (int e = 0; e < 4; ++e) bv[cb][i][e] = in ? bv[cb][i][e] : 0u;
                }
                cv[cb] = kb + 32 * lg < K ? cv[cb] : 0.f;
            }
        }
        f32x4_t c0[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            c0[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(cv[cb], -1.0f, f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) {
            half8_t B[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t x = wv[rt][i], y = x >> 8;
                u32x4 av;
                av[0] = and_or_u32(0x000F000Fu, x, magic);
                av[1] = and_or_u32(0x00F000F0u, x, magic);
                av[2] = and_or_u32(0x000F000Fu, y, magic);
                av[3] = and_or_u32(0x00F000F0u, y, magic);
                B[i] = __builtin_bit_cast(half8_t, av);
            }
            const float scl = f16_to_f32(sv[rt]);
            f32x4_t c[NCB];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
                    c[cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, bv[cb][i]), B[i], i == 0 ? c0[cb] : c[cb], 0, 0, 0);
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[rt][cb][j] = __builtin_fmaf(scl, c[cb][j], acc[rt][cb][j]);
        }
    };
    // each tile starts its range at its own group (rotation by the tile's index, in
    // a matrix that may run in pairs by the pair's, for either PT: the order of the
    // sums, and with it the result, must not depend on the form): at
    // any moment the workgroups read different parts of the prepared operand
    const int n = g1 - g0, rot = __builtin_amdgcn_readfirstlane(n > 0 ? (a.pair_rot ? t >> 1 : t) % n : 0);
    auto G = [&](int q) {
        q = min(q, n - 1) + rot;
        return g0 + (q >= n ? q - n : q);
    };
    // With 17 or more rows the residual epilogue's inputs (the tile's residual
    // rows, the next norm's weights and the rows' rs) are read now by every split
    // of the tile, off the last split's tail; the residual is rewritten only by
    // the tile's last split to arrive, after all have started.  (With 16 rows the
    // added start latency outweighs the shorter tail: measured.)
    const bool resid_epi = PRE && a.epi == EPI_RESID;
    float pres[NV], prs = 0.f;
    uint16_t pgam_bits = 0;
    if (resid_epi) {
        size_t off[NV];                                  // clamped to a valid element; outside rows are never used
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q, m = min(m0 + (idx >> 6), M - 1), n = min(t * 64 + (idx & 63), W.n - 1);
            off[q] = (size_t)m * a.resid_ld + n;
        }
        load_vals(a.resid, a.resid_dt, off, pres);
        if (a.bp_out) {                                  // raw now, converted once every load is out
            pgam_bits = a.gamma_next[min(t * 64 + (tid & 63), W.n - 1)];
            prs = a.rs_in[min(m0 + tid, M - 1)];
        }
    }
    // factor of each row (rs / c for a deferred RMSNorm input, else 1): its
    // inputs come from the kernel before; they and the epilogue's inputs are
    // issued before the first group's loads, so nothing below waits for those
    RowFactorLoads rfl;
    row_factor_loads(a, rfl);
    __builtin_amdgcn_sched_barrier(0);
    if (n > 0) {
        ldw(G(0), wr[0], sr[0]);
        if constexpr (PT == 1) ldb(G(0), br[0], cr[0]);
        else {
            ldc(G(0), cr[0]);
            ldh(G(0));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    row_factors_finish(a, K, t == 0 && s == 0, rfl, fs);
    if constexpr (PRE) {
        if (resid_epi) {
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const int idx = tid + 256 * q;
                sres[idx >> 6][idx & 63] = pres[q];
            }
            if (tid < 64) sgam[tid] = half_bits_to_f32(pgam_bits, a.gamma_next_dt);
            if (tid < MP) srs[tid] = prs;
        }
    }
    if constexpr (PT == 2) {
        // step q: the K range's rows of group q are in LDS buffer q & 1; every wave
        // takes kg steps (the barriers), those past its range without products
        if (n > 0) {
            puth(0);
            ldh(G(1));
        }
        auto step = [&](int q, u32x4 (&wv)[4], uint16_t (&sv)[4], float (&cv)[NCB], u32x4 (&wn)[4], uint16_t (&sn)[4], float (&cn)[NCB]) {
            __syncthreads();
            if (q >= n) return;                          // uniform in the wave
            ldw(G(q + 1), wn, sn);
            ldc(G(q + 1), cn);
            puth((q + 1) & 1);
            ldh(G(q + 2));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int i = 0; i < 4; ++i) br[0][cb][i] = sb[q & 1][w][4 * cb + i][lane];
            compute(G(q), wv, sv, br[0], cv);
        };
        for (int q = 0; q < a.kg; q += 2) {
            step(q, wr[0], sr[0], cr[0], wr[1], sr[1], cr[1]);
            if (q + 1 < a.kg) step(q + 1, wr[1], sr[1], cr[1], wr[0], sr[0], cr[0]);
        }
        __syncthreads();                                 // the rows in LDS give way to the sums
    } else if (n > 0) {
        // group q computes from set q & 1 while group q + 1 loads into the other set:
        // whole pairs of groups, then a last single group
        int q = 0;
        for (; q + 2 <= n; q += 2) {
            ldw(G(q + 1), wr[1], sr[1]);
            ldb(G(q + 1), br[1], cr[1]);
            __builtin_amdgcn_sched_barrier(0);           // the loads issue before this group's products
            compute(G(q), wr[0], sr[0], br[0], cr[0]);
            ldw(G(q + 2), wr[0], sr[0]);
            ldb(G(q + 2), br[0], cr[0]);
            __builtin_amdgcn_sched_barrier(0);
            compute(G(q + 1), wr[1], sr[1], br[1], cr[1]);
        }
        if (q < n) {
            ldw(G(q + 1), wr[1], sr[1]);
            ldb(G(q + 1), br[1], cr[1]);
            __builtin_amdgcn_sched_barrier(0);
            compute(G(q), wr[0], sr[0], br[0], cr[0]);
        }
    }
    // ---- the 4 waves' sums of each output (lane: weight row 16 rt + l16 of input rows 16 cb + 4 lg + j), in wave order
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[w][16 * cb + 4 * lg + j][16 * rt + l16] = acc[rt][cb][j];
    __syncthreads();
    float vals[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int idx = tid + 256 * q, m = idx >> 6, r = idx & 63;
        vals[q] = (red[0][m][r] + red[1][m][r]) + (red[2][m][r] + red[3][m][r]);
    }

    // ---- split-K: the last workgroup of the tile sums every split in split order
    if (PT == 1 && a.ksplit > 1) {
        const int ldp = W.ntiles * 64;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (m0 + (idx >> 6) < M)
                store_coherent(&a.partial[((size_t)s * M + m0 + (idx >> 6)) * ldp + t * 64 + (idx & 63)], vals[q]);
        }
        if (!last_arrival(&a.counters[Z == 1 ? t : 2 * t + (m0 >> 5)], (unsigned)a.ksplit, &last_s)) return;
        const size_t stride = (size_t)M * ldp;
#pragma unroll
        for (int q = 0; q < NV; ++q) vals[q] = 0.f;
        for (int s0 = 0; s0 < a.ksplit; s0 += 4) {
            float b4[NV][4];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const int idx = tid + 256 * q;
                const float* pp = &a.partial[(size_t)(m0 + (idx >> 6)) * ldp + t * 64 + (idx & 63)];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    b4[q][e] = (m0 + (idx >> 6) < M && s0 + e < a.ksplit) ? load_coherent(pp + (s0 + e) * stride) : 0.f;
            }
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) vals[q] += b4[q][e];
        }
    }

    // ---- epilogue (row limit 0 for a missing tile: its threads only take part in the barriers and sums)
    const int Mt = has ? M : 0;
    if (a.epi == EPI_STORE) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (m0 + (idx >> 6) < Mt) {
                const int m = m0 + (idx >> 6), n = t * 64 + (idx & 63);
                if (n < W.n) a.out[(size_t)m * a.out_ld + n] = vals[q] * fs[m];
            }
        }
    } else if (PT == 1 && a.epi == EPI_RESID) {
        // the residual rows, the next norm's weights and the rows' rs (read at the
        // start with 17 or more rows), every load issued before any is used
        float xres[NV], egam[NV], ers[NV];
        if constexpr (!PRE) {
            size_t off[NV];
            uint16_t gbits[NV];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const int idx = tid + 256 * q, m = min(m0 + (idx >> 6), M - 1), n = min(t * 64 + (idx & 63), W.n - 1);
                off[q] = (size_t)m * a.resid_ld + n;
                gbits[q] = a.bp_out ? a.gamma_next[n] : (uint16_t)0;
                ers[q] = a.bp_out ? a.rs_in[m] : 0.f;
            }
            load_vals(a.resid, a.resid_dt, off, xres);
#pragma unroll
            for (int q = 0; q < NV; ++q) egam[q] = half_bits_to_f32(gbits[q], a.gamma_next_dt);
        }
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            const int m = m0 + (idx >> 6), r = idx & 63;              // one row per wave: whole waves take part
            const int n = t * 64 + r;
            const bool ok = m < M && n < W.n;
            float xn = 0.f;
            if (ok) {
                float xr;
                if constexpr (PRE) xr = sres[m - m0][r];
                else xr = xres[q];
                xn = xr + vals[q] * fs[m];
                a.out[(size_t)m * a.out_ld + n] = xn;
                if (a.out_act) ((uint16_t*)a.out_act)[(size_t)m * a.out_act_ld + n] = to_half_bits(xn, a.out_act_dt);
            }
            // the row's sum of squares over the tile: row m is this wave's 64 lanes
            const float ss = wave_sum_all(xn * xn);
            if (a.ssq_out && m < M && r == 0) a.ssq_out[(size_t)m * W.ntiles + t] = ss;
            if (a.bp_out && m < M) {                                    // the next product's input
                float c, gm;
                if constexpr (PRE) {
                    c = srs[m - m0];
                    gm = sgam[r];
                } else {
                    c = ers[q];
                    gm = egam[q];
                }
                const float h = ok ? xn * gm * c : 0.f;
                bp_put(a.bp_out, a.bc_out, a.kp, m, n, h, ok);
                if (t == 0 && r == 0) a.cb_out[m] = c;
            }
        }
    } else if (a.epi == EPI_TOP1) {
        // per row: the tile's largest value, its smallest index among equal ones,
        // and the sum of exp(v - max) over the tile (row m is one wave's 64 lanes)
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            const int m = m0 + (idx >> 6), r = idx & 63;
            if (m >= Mt) continue;                                     // uniform in the wave
            const int n = t * 64 + r;
            const bool ok = n < W.n;
            const float v = ok ? vals[q] * fs[m] : -INFINITY;
            if (ok && a.out) a.out[(size_t)m * a.out_ld + n] = v;
            const float mx = wave_max_all(v);
            const int arg = wave_min_all((ok && v == mx) ? n : INT_MAX);
            const float se = wave_sum_all(ok ? expf(v - mx) : 0.f);
            if (r == 0) a.top1_part[(size_t)m * W.ntiles + t] = make_float4(mx, __int_as_float(arg), se, 0.f);
        }
    } else {  // EPI_SWIGLU: rows 0..31 of the tile are gate rows, 32..63 the matching up rows
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + 256 * q;
            if (m0 + (idx >> 6) < M) red[0][idx >> 6][idx & 63] = vals[q] * fs[m0 + (idx >> 6)];
        }
        __syncthreads();
        for (int i0 = 0; i0 < MP * 32; i0 += 256) {                    // whole waves: two rows each
            const int idx = i0 + tid;
            const int ml = idx >> 5, m = m0 + ml, r = idx & 31;
            const int f = t * 32 + r;
            const bool ok = m < Mt && f < a.n_valid;
            float y = 0.f;
            if (ok) {
                const float gt = red[0][ml][r], up = red[0][ml][r + 32];
                y = (gt / (1.0f + expf(-gt))) * up;
                a.out[(size_t)m * a.out_ld + f] = y;
            }
            if (a.bp_out && m < Mt) bp_put(a.bp_out, a.bc_out, a.kp, m, f, y, ok);
        }
    }
}

hipError_t launch_gemm_bp(const GemvArgs& a, hipStream_t st) {
    if (a.M < 1 || a.M > 64 || a.W.gchunks != 4 || a.kg < 1 || a.kp % 128) return hipErrorInvalidValue;
    // two tiles per workgroup: more than 16 rows, both tiles' groups in the pair's
    // order, whole sums, no residual
    if (a.pt != 1 && (a.pt != 2 || a.M <= 16 || !a.pair_rot || a.ksplit != 1 || a.epi == EPI_RESID)) return hipErrorInvalidValue;
    const int wgs = (a.W.ntiles + a.pt - 1) / a.pt;
    const dim3 grid(wgs, a.ksplit), zgrid((wgs + 7) / 8 * 16, a.ksplit), block(256 * a.pt);
    if (a.pt == 1) {
        if (a.M <= 16) gemm_bp_kernel<1, 1, 1><<<grid, block, 0, st>>>(a);
        else if (a.M <= 32) gemm_bp_kernel<2, 1, 1><<<grid, block, 0, st>>>(a);
        else gemm_bp_kernel<2, 2, 1><<<zgrid, block, 0, st>>>(a);
    } else {
        if (a.M <= 32) gemm_bp_kernel<2, 1, 2><<<grid, block, 0, st>>>(a);
        else gemm_bp_kernel<2, 2, 2><<<zgrid, block, 0, st>>>(a);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ prefill product

// Eight consecutive values at element offset i of p (fp32 at 16-byte aligned
// offsets; 16-bit values at any 2-byte aligned address).
__device__ __forceinline__ void load8(const void* p, int dt, size_t i, float (&v)[8]) {
    if (dt == DT_F32) {
        float4 x[2];
        x[0] = *(const float4*)((const float*)p + i);
        x[1] = *(const float4*)((const float*)p + i + 4);
        __builtin_memcpy(v, x, 32);
    } else {
        uint16_t h[8];
        __builtin_memcpy(h, (const uint16_t*)p + i, 16);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = dt == DT_BF16 ? bf16_to_f32(h[e]) : f16_to_f32(h[e]);
    }
}

// Rows of a prompt: x = in + the splits of a product (added in split order; to
// x_out, and to out_act in the act dtype); then RMSNorm(x) * gamma as the
// prepared input of the next product, row r as row r mod 64 of block r / 64.
// One wave per row, eight rows per workgroup (the eight 16-byte pieces a 128-byte
// line of a block takes come from one workgroup), eight consecutive k per lane
// and step; the row stays in registers up to 512 NS values (NS = 0: it is read
// again, for longer rows).  Bound by memory latency at few rows (517 x 4096 with
// 3 splits 17 us), by traffic at many (2048 x 4096: 39 -> 14 us, 3.5 TB/s).
template <int NS>
__global__ __launch_bounds__(512) void bprep_rows_kernel(PfRows a) {
    const int lane = threadIdx.x & 63, r = 8 * blockIdx.x + (threadIdx.x >> 6);
    if (r >= a.n) return;                                      // waves are independent: no barrier below
    const int K = a.K;
    auto load = [&](int k, float (&v)[8]) {
        load8(a.in, a.in_dt, (size_t)r * a.in_ld + k, v);
        for (int s = 0; s < a.nsplit; ++s) {
            float p[8];
            load8(a.part, DT_F32, (size_t)s * a.part_stride + (size_t)r * K + k, p);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += p[e];
        }
    };
    auto put_x = [&](int k, const float (&v)[8]) {
        if (a.x_out) __builtin_memcpy(a.x_out + (size_t)r * K + k, v, 32);
        if (a.out_act) {
            uint16_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = to_half_bits(v[e], a.out_act_dt);
            __builtin_memcpy((uint16_t*)a.out_act + (size_t)r * K + k, h, 16);
        }
    };
    float x[NS ? NS : 1][8];
    float ss = 0.f;
    if constexpr (NS > 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = 512 * s + 8 * lane;
#pragma unroll
            for (int e = 0; e < 8; ++e) x[s][e] = 0.f;
            if (k < K) load8(a.in, a.in_dt, (size_t)r * a.in_ld + k, x[s]);
        }
        for (int sp = 0; sp < a.nsplit; ++sp) {
            const float* pr = a.part + (size_t)sp * a.part_stride + (size_t)r * K + 8 * lane;
#pragma unroll
            for (int h = 0; h < NS; h += 8) {                  // eight steps' loads at once
                float p[8][8];
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    if (512 * (h + s) + 8 * lane < K) load8(pr, DT_F32, 512 * (h + s), p[s]);
#pragma unroll
                for (int s = 0; s < 8; ++s)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (512 * (h + s) + 8 * lane < K) x[h + s][e] += p[s][e];
            }
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = 512 * s + 8 * lane;
            if (k < K) put_x(k, x[s]);
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += x[s][e] * x[s][e];
        }
    } else {
        for (int k = 8 * lane; k < K; k += 512) {
            load(k, x[0]);
            put_x(k, x[0]);
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += x[0][e] * x[0][e];
        }
    }
    if (!a.bp) return;
    const float rs = rsqrtf(wave_sum_all(ss) / (float)K + a.eps);
    uint16_t* bp = a.bp + (size_t)(r >> 6) * 64 * a.kp;
    float* bc = a.bc + (size_t)(r >> 6) * 2 * a.kp;
    auto prep = [&](int k, const float (&v)[8]) {
        const bool in = k < K;
        float g[8];
        load8(a.gamma, a.gamma_dt, min(k, K - 8), g);
        uint16_t c[8];
        float cs = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float h16 = f16_to_f32(f32_to_f16(v[e] * rs * g[e]));
            cs += bp_corr(h16, e);
            c[e] = bp_code(h16, e);
        }
        cs = in ? cs : 0.f;
        cs += dpp_f<0xB1>(cs);
        cs += dpp_f<0x4E>(cs);                                 // the 4 lanes of 32 k
        if (in) {
            __builtin_memcpy(__builtin_assume_aligned(bp + bp_index(r & 63, k), 16), c, 16);
            if ((k & 31) == 0) bc[bc_index(r & 63, k)] = cs;
        }
    };
    if constexpr (NS > 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (512 * s < K) prep(512 * s + 8 * lane, x[s]);   // whole waves take part in the sums
    } else {
        for (int k0 = 0; k0 < K; k0 += 512) {
            const int k = k0 + 8 * lane, kc = min(k, K - 8);
            if (a.x_out) load8(a.x_out, DT_F32, (size_t)r * K + kc, x[0]);
            else load(kc, x[0]);
            prep(k, x[0]);
        }
    }
}

hipError_t launch_bprep_rows(const PfRows& a, hipStream_t st) {
    if (a.K < 8 || a.K % 8 || a.n < 1 || (a.bp && (a.kp < a.K || a.kp % 128))) return hipErrorInvalidValue;
    const dim3 grid((a.n + 7) / 8), block(512);
    if (a.K <= 4096) bprep_rows_kernel<8><<<grid, block, 0, st>>>(a);
    else if (a.K <= 8192) bprep_rows_kernel<16><<<grid, block, 0, st>>>(a);
    else bprep_rows_kernel<0><<<grid, block, 0, st>>>(a);
    return hipGetLastError();
}

// Product of a prompt's prepared rows with one matrix.  A workgroup takes four
// 64-row weight tiles (one per wave) and one 64-token block, over all of K.
// Per group of 128 k the block's 16 operand fragments (16 KB) go through
// registers into LDS (two buffers) and are shared by the four waves; each wave
// decodes its tile's codes into matrix-core operands as gemm_bp_kernel does.
// The products are taken transposed (tokens as the rows, weight rows as the
// columns): a lane's results are four tokens of one weight row, so a row's
// scale is one register, and the corrections of four tokens are the products'
// starting value (one 16-byte LDS read), which leaves one multiply-add per
// result and group.  The next group's codes and the one after's fragments are
// in flight while a group computes.
// Bound by issue: per 64 products a wave also issues about 165 vector
// instructions (80 decode, 64 scale), and products and vector instructions of
// the two waves of a SIMD overlap only in part (matrix cores busy half the time,
// at about 1.8 GHz).  gate|up of 2048 tokens (8B) 622 -> 456 us, 1.05 PFLOP/s
// (a large fp16 library product reaches 1.16 on this card).
// RAG: K is not a multiple of 128 (operand entries past K are dropped).
template <bool RAG>
__global__ __launch_bounds__(256, 2) void gemm_pf_kernel(PfArgs a) {
    __shared__ __attribute__((aligned(16))) u32x4 sb[2][16][64];
    __shared__ __attribute__((aligned(16))) float sc[2][64];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    // workgroups of one XCD (blockIdx mod 8) walk the tiles in bands of PF_BAND
    // token blocks: the 64 that run at once share 8 weight tile groups and 8
    // token blocks in the XCD's L2
    const int tiles = a.nwt * a.ntb, total = tiles * a.ksplit;
    const int per_xcd = (total + 7) / 8;
    int q = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || q >= total) return;   // whole workgroup: no barrier is reached
    const int s = q / tiles;                                   // split of K
    q -= s * tiles;
    const int band = q / (PF_BAND * a.nwt), inb = q - band * PF_BAND * a.nwt;
    const int bw = min(PF_BAND, a.ntb - band * PF_BAND);
    const int wt = inb / bw, tb = band * PF_BAND + inb % bw;
    const PackedMat W = a.W;
    const int t = 4 * wt + w;
    const bool has = t < W.ntiles;
    const int tt = has ? t : W.ntiles - 1;                     // loads stay in bounds; results are dropped
    const int K = W.k;
    const int g0 = s * a.kg, ng = min((K + 127) / 128, g0 + a.kg);   // this split's groups: g0 .. ng - 1
    // buffer resources: uniform group offsets, one 32-bit offset per lane
    const __amdgpu_buffer_rsrc_t rbp = buf_rsrc(a.bp + (size_t)tb * a.bp_blk, (uint32_t)a.bp_blk * 2);
    const __amdgpu_buffer_rsrc_t rbc = buf_rsrc(a.bc + (size_t)tb * a.bc_blk, (uint32_t)a.bc_blk * 4);
    const __amdgpu_buffer_rsrc_t rw = buf_rsrc(W.w + (size_t)tt * W.nchunk * 1024, (uint32_t)W.nchunk * 1024);
    const __amdgpu_buffer_rsrc_t rs = buf_rsrc(W.s + (size_t)tt * W.ngroups * 64, (uint32_t)W.ngroups * 128);
    const uint32_t bo = 16u * tid, co = 4u * tid, wo = 16u * (64 * lg + l16), so = 2u * l16;
    uint32_t magic = 0x64006400u;
    asm volatile("" : "+v"(magic));

    u32x4 rb[4];
    float rc;
    // one group's operand fragments (fragment 4 u + w by wave w) and corrections
    // (thread 4 r + c: chunk c of token r)
    auto ld_b = [&](int g) {
#pragma unroll
        for (int u = 0; u < 4; ++u) rb[u] = buf_load16(rbp, bo, 16384 * g + 4096 * u);
        rc = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rbc, co, 1024 * g, 0));
    };
    auto st_b = [&](int g) {
        const int buf = g & 1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            u32x4 v = rb[u];
            if constexpr (RAG) {                               // fragment f = 4 cb + i holds k = 32 lg + 8 i + e
                const bool in = 128 * g + 32 * lg + 8 * w < K;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = in ? v[e] : 0u;
            }
            sb[buf][4 * u + w][lane] = v;
        }
        float s = rc;
        if constexpr (RAG) s = 128 * g + 32 * (tid & 3) < K ? s : 0.f;
        s += dpp_f<0xB1>(s);                                   // lane ^ 1
        s += dpp_f<0x4E>(s);                                   // lane ^ 2: the token's 4 chunks
        sc[buf][tid >> 2] = -s;                                // the same value from 4 lanes
    };
    u32x4 cw[4];
    uint16_t cs[4];
    auto ld_w = [&](int g, int rt) {
        cw[rt] = buf_load16(rw, wo, 4096 * g + 256 * rt);
        cs[rt] = __builtin_amdgcn_raw_buffer_load_b16(rs, so, 128 * g + 32 * rt, 0);
    };
    auto decode = [&](const u32x4& v, half8_t (&B)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t x = v[i], y = x >> 8;
            u32x4 av;
            av[0] = and_or_u32(0x000F000Fu, x, magic);
            av[1] = and_or_u32(0x00F000F0u, x, magic);
            av[2] = and_or_u32(0x000F000Fu, y, magic);
            av[3] = and_or_u32(0x00F000F0u, y, magic);
            B[i] = __builtin_bit_cast(half8_t, av);
        }
    };

    f32x4_t acc[4][4], c[2][4];
    half8_t A[4][4], B[2][4];
    float scl[2];
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) acc[rt][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    ld_b(g0);
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) ld_w(g0, rt);
    st_b(g0);
    ld_b(min(g0 + 1, ng - 1));
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
        for (int i = 0; i < 4; ++i) A[cb][i] = __builtin_bit_cast(half8_t, sb[g0 & 1][4 * cb + i][lane]);
        c[0][cb] = *(const f32x4_t*)&sc[g0 & 1][16 * cb + 4 * lg];
        c[1][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    decode(cw[0], B[0]);
    scl[0] = f16_to_f32(cs[0]);
    scl[1] = 0.f;
    ld_w(min(g0 + 1, ng - 1), 0);
    // One group in four steps of one 16-row weight block: 16 products, k slice by
    // k slice over four independent token blocks.  While a step's products run, the
    // step before's results are scaled into the sums and its registers reloaded with
    // the next starting values, and the next step's codes are decoded (and their
    // registers reloaded with the next group's).  Step 1 fills the other LDS buffer;
    // the barrier at step 3 opens it (by then every wave holds all of this group's
    // operands and corrections), and step 3 replaces each token operand after its
    // last product.  Past the last group the loads repeat it and what they feed is
    // not used.
    for (int g = g0; g < ng; ++g) {
        const int buf = g & 1, gn = min(g + 1, ng - 1);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) {
            const int p = rt & 1;
            __builtin_amdgcn_sched_barrier(0);
            if (rt == 1) {
                st_b(g + 1);
                ld_b(min(g + 2, ng - 1));
            }
            if (rt == 3) __syncthreads();
            decode(cw[(rt + 1) & 3], B[p ^ 1]);
            const float sp = scl[p ^ 1];
            scl[p ^ 1] = f16_to_f32(cs[(rt + 1) & 3]);
            ld_w(rt < 3 ? gn : min(g + 2, ng - 1), (rt + 1) & 3);
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[(rt + 3) & 3][cb][j] = __builtin_fmaf(sp, c[p ^ 1][cb][j], acc[(rt + 3) & 3][cb][j]);
                c[p ^ 1][cb] = *(const f32x4_t*)&sc[rt < 3 ? buf : buf ^ 1][16 * cb + 4 * lg];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    c[p][cb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[cb][i], B[p][i], c[p][cb], 0, 0, 0);
                    if (rt == 3) A[cb][i] = __builtin_bit_cast(half8_t, sb[buf ^ 1][4 * cb + i][lane]);
                }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            }
        }
    }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[3][cb][j] = __builtin_fmaf(scl[1], c[1][cb][j], acc[3][cb][j]);
    // ---- epilogue: lane holds row 64 t + 16 rt + l16 of tokens 64 tb + 16 cb + 4 lg + j
    if (a.epi == EPI_SWIGLU) {
        // rows 0..31 of a tile gate, 32..63 the matching up: the workgroup's four
        // tiles give one whole group of 128 values of the down product's input,
        // written in prepared form (wave w: chunk w) through LDS as 16 KB in a row.
        // Values past n_valid are zero.
        __syncthreads();                                        // the operands in sb are no longer read
        uint16_t* sy = (uint16_t*)&sb[0][0][0];
        float* bco = a.bc_out + (size_t)tb * a.out_bc_blk + (size_t)wt * 256 + w;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m = 16 * cb + 4 * lg + j;
                float cs = 0.f;
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    const int f = 32 * t + 16 * rt + l16;
                    const float gt = acc[rt][cb][j], up = acc[rt + 2][cb][j];
                    const float y = has && f < a.n_valid ? (gt / (1.0f + expf(-gt))) * up : 0.f;
                    const float h16 = f16_to_f32(f32_to_f16(y));
                    cs += bp_corr(h16, l16);
                    sy[((4 * cb + 2 * rt + (l16 >> 3)) * 64 + 16 * w + 4 * lg + j) * 8 + (l16 & 7)] = bp_code(h16, l16);
                }
                cs = sum16(cs);
                if (l16 == 0) bco[4 * m] = cs;
            }
        __syncthreads();
        u32x4* bpo = (u32x4*)(a.bp_out + (size_t)tb * a.out_bp_blk) + (size_t)wt * 1024 + tid;
#pragma unroll
        for (int u = 0; u < 4; ++u) bpo[256 * u] = (&sb[0][0][0])[tid + 256 * u];
        return;
    }
    if (!has) return;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int tok = 64 * tb + 16 * cb + 4 * lg + j;
            if (tok >= a.n) continue;
#pragma unroll
            for (int rt = 0; rt < 4; ++rt) {
                const int row = 64 * t + 16 * rt + l16;
                if (row >= W.n) continue;
                float v = acc[rt][cb][j];
                if (a.ksplit > 1) {                            // this split's sums; the next bprep_rows_kernel adds them
                    a.part[(size_t)s * a.part_stride + (size_t)tok * a.out_ld + row] = v;
                    continue;
                }
                if (a.epi == EPI_RESID) {
                    v += load_val(a.resid, a.resid_dt, (size_t)tok * a.resid_ld + row);
                    if (a.out_act) ((uint16_t*)a.out_act)[(size_t)tok * a.out_act_ld + row] = to_half_bits(v, a.out_act_dt);
                }
                a.out[(size_t)tok * a.out_ld + row] = v;
            }
        }
}

hipError_t launch_gemm_pf(const PfArgs& a, hipStream_t st) {
    if (a.n < 1 || a.W.gchunks != 4 || a.nwt != (a.W.ntiles + 3) / 4 || a.ntb != (a.n + 63) / 64) return hipErrorInvalidValue;
    const int ng = (a.W.k + 127) / 128;                        // every split holds at least one group
    if (a.ksplit < 1 || a.kg < 1 || a.ksplit * a.kg < ng || (a.ksplit - 1) * a.kg >= ng) return hipErrorInvalidValue;
    if (a.ksplit > 1 && (!a.part || a.epi != EPI_RESID)) return hipErrorInvalidValue;
    const int total = a.nwt * a.ntb * a.ksplit;
    const unsigned grid = 8u * (unsigned)((total + 7) / 8);
    if (a.W.k % 128) gemm_pf_kernel<true><<<dim3(grid), dim3(256), 0, st>>>(a);
    else gemm_pf_kernel<false><<<dim3(grid), dim3(256), 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_bprep(const void* in, int in_dt, int in_ld, const uint16_t* gamma, int gamma_dt, int K, float eps,
                        int M, uint16_t* bp, float* bc, int kp, float* rs_out, hipStream_t st) {
    if (K < 1 || K > 32 * 256) return hipErrorInvalidValue;
    bprep_kernel<<<dim3(M, (K + BPREP_SLICE - 1) / BPREP_SLICE), 256, 0, st>>>(in, in_dt, in_ld, gamma, gamma_dt, K, eps,
                                                                              bp, bc, kp, rs_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ attention

// Rows [j0, j1) of one split are processed in blocks of ABLK keys whose mask
// bytes and table entries are first staged in LDS; each 16-lane key group then
// loads KB cache rows at once before scoring them.
constexpr int ABLK = 256;
constexpr int KB = 4;

template <int D, int RC>
__global__ __launch_bounds__(256) void attn_kernel(AttnArgs a) {
    constexpr int EPL = D / 16;
    constexpr int HALF = D / 2;
    __shared__ float lo[KGROUPS][RC][D];
    __shared__ float lm[KGROUPS][RC], ll[KGROUPS][RC];
    __shared__ uint8_t smask[ABLK];
    __shared__ int16_t stab[ABLK];

    const int item = blockIdx.x, g = blockIdx.y, split = blockIdx.z;
    const ItemDev it = a.meta.items[item];
    const ReqDev rq = it.rq;
    const int b = it.slot;
    const int P = rq.P, n = rq.n;
    const int L = P + n;
    const int split_len = rq.split_len;
    const int nsplit = (L + split_len - 1) / split_len;
    if (split >= nsplit) return;
    const int j0 = split * split_len, j1 = min(L, j0 + split_len);

    const int tid = threadIdx.x, kg = tid >> 4, li = tid & 15;
    const int Hq = a.Hq, Hkv = a.Hkv;
    const int gs = Hq / Hkv;
    const int R = gs * n;
    const size_t lstride = (size_t)rq.S * Hkv * rq.cap * D;
    uint16_t* kl = rq.kc + (size_t)a.layer * lstride;
    uint16_t* vl = rq.vc + (size_t)a.layer * lstride;
    const uint8_t* mask = a.meta.masks + rq.mask_off + (size_t)b * rq.mask_len;
    // per-query-row masks of the slot, [n][mask_len], when the request has them
    const uint8_t* rmask = rq.rowmask_off >= 0 ? a.meta.masks + rq.rowmask_off + (size_t)b * n * rq.mask_len : nullptr;
    const int16_t* tab = rq.table + (size_t)b * rq.cap;
    const int rowbase = rq.row0 + b * n;
    const int d0 = li * EPL;
    const int jc1 = min(j1, P);            // cached rows end here; [max(j0, P), j1) are new rows

    for (int r0 = 0; r0 < R; r0 += RC) {
        float q[RC][EPL];
        int qi[RC];
#pragma unroll
        for (int rr = 0; rr < RC; ++rr) {
            const int r = r0 + rr;
            qi[rr] = -1;
#pragma unroll
            for (int e = 0; e < EPL; ++e) q[rr][e] = 0.f;
            if (r < R) {
                const int i = r / gs, h = g * gs + (r % gs);
                const int m = rowbase + i;
                const int pos = a.meta.positions[m];
                const float* qrow = a.qkv + (size_t)m * a.qkv_ld + (size_t)h * D;
                qi[rr] = i;
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    const int d = d0 + e;
                    const bool lo_half = d < HALF;
                    const float x = qrow[d];
                    const float xp = lo_half ? qrow[d + HALF] : qrow[d - HALF];
                    const float2 cs = a.rope[(size_t)pos * HALF + (lo_half ? d : d - HALF)];
                    const float y = lo_half ? (x * cs.x - xp * cs.y) : (x * cs.x + xp * cs.y);
                    q[rr][e] = y * a.qscale;
                }
            }
        }
        float mx[RC], sl[RC], o[RC][EPL];
#pragma unroll
        for (int rr = 0; rr < RC; ++rr) {
            mx[rr] = -INFINITY;
            sl[rr] = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) o[rr][e] = 0.f;
        }

        auto consume = [&](int j, const float* kf, const float* vf) {
#pragma unroll
            for (int rr = 0; rr < RC; ++rr) {
                if (qi[rr] < 0) continue;
                float sd = 0.f;
#pragma unroll
                for (int e = 0; e < EPL; ++e) sd += q[rr][e] * kf[e];
                sd = sum16(sd);
                if (j > P + qi[rr]) continue;                 // causal over the physical index
                if (rmask && rmask[(size_t)qi[rr] * rq.mask_len + j] == 0) continue;   // hidden from this row
                const float mn = fmaxf(mx[rr], sd);
                const float corr = exp2f(mx[rr] - mn);
                const float p = exp2f(sd - mn);
                sl[rr] = sl[rr] * corr + p;
#pragma unroll
                for (int e = 0; e < EPL; ++e) o[rr][e] = o[rr][e] * corr + p * vf[e];
                mx[rr] = mn;
            }
        };

        // ---- cached rows: read through the beam table
        for (int jb = j0; jb < jc1; jb += ABLK) {
            const int nb = min(ABLK, jc1 - jb);
            __syncthreads();
            for (int x = tid; x < nb; x += 256) {
                smask[x] = mask[jb + x];
                stab[x] = tab[jb + x];
            }
            __syncthreads();
            for (int x0 = kg; x0 < nb; x0 += KGROUPS * KB) {
                uint16_t kb[KB][EPL], vb[KB][EPL];
                bool vis[KB];
#pragma unroll
                for (int u = 0; u < KB; ++u) {
                    const int x = x0 + u * KGROUPS;
                    vis[u] = (x < nb) && smask[x] != 0;      // hidden from every query of the slot
                    if (vis[u]) {
                        const int j = jb + x;
                        const size_t off = (((size_t)stab[x] * Hkv + g) * rq.cap + j) * D + d0;
                        if constexpr (EPL == 8) {
                            *(u32x4*)kb[u] = *(const u32x4*)(kl + off);
                            *(u32x4*)vb[u] = *(const u32x4*)(vl + off);
                        } else {
                            *(u32x2*)kb[u] = *(const u32x2*)(kl + off);
                            *(u32x2*)vb[u] = *(const u32x2*)(vl + off);
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < KB; ++u) {
                    if (!vis[u]) continue;
                    float kf[EPL], vf[EPL];
#pragma unroll
                    for (int e = 0; e < EPL; ++e) {
                        kf[e] = half_bits_to_f32(kb[u][e], a.kv_dt);
                        vf[e] = half_bits_to_f32(vb[u][e], a.kv_dt);
                    }
                    consume(jb + x0 + u * KGROUPS, kf, vf);
                }
            }
        }

        // ---- this forward's rows: rotate k, round k and v to the cache dtype, append
        for (int j = max(j0, P) + kg; j < j1; j += KGROUPS) {
            if (mask[j] == 0) continue;
            const int i = j - P;
            const int m = rowbase + i;
            const int pos = a.meta.positions[m];
            const float* krow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + g) * D;
            const float* vrow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + Hkv + g) * D;
            uint16_t kb[EPL], vb[EPL];
            float kf[EPL], vf[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                const int d = d0 + e;
                const bool lo_half = d < HALF;
                const float x = krow[d];
                const float xp = lo_half ? krow[d + HALF] : krow[d - HALF];
                const float2 cs = a.rope[(size_t)pos * HALF + (lo_half ? d : d - HALF)];
                const float y = lo_half ? (x * cs.x - xp * cs.y) : (x * cs.x + xp * cs.y);
                kb[e] = to_half_bits(y, a.kv_dt);
                vb[e] = to_half_bits(vrow[d], a.kv_dt);
                kf[e] = half_bits_to_f32(kb[e], a.kv_dt);
                vf[e] = half_bits_to_f32(vb[e], a.kv_dt);
            }
            consume(j, kf, vf);
        }
        if (r0 == 0 && !a.no_append) {          // append: owner of row j writes it
            for (int j = max(j0, P) + kg; j < j1; j += KGROUPS) {
                const int i = j - P;
                const int m = rowbase + i;
                const int pos = a.meta.positions[m];
                const float* krow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + g) * D;
                const float* vrow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + Hkv + g) * D;
                const size_t off = (((size_t)b * Hkv + g) * rq.cap + j) * D + d0;
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    const int d = d0 + e;
                    const bool lo_half = d < HALF;
                    const float x = krow[d];
                    const float xp = lo_half ? krow[d + HALF] : krow[d - HALF];
                    const float2 cs = a.rope[(size_t)pos * HALF + (lo_half ? d : d - HALF)];
                    const float y = lo_half ? (x * cs.x - xp * cs.y) : (x * cs.x + xp * cs.y);
                    kl[off + e] = to_half_bits(y, a.kv_dt);
                    vl[off + e] = to_half_bits(vrow[d], a.kv_dt);
                }
                if (a.layer == 0 && g == 0 && li == 0) rq.table[(size_t)b * rq.cap + j] = (int16_t)b;
            }
        }

        // ---- merge the 16 key groups (fixed order) into this split's partial
#pragma unroll
        for (int rr = 0; rr < RC; ++rr) {
            if (li == 0) {
                lm[kg][rr] = mx[rr];
                ll[kg][rr] = sl[rr];
            }
#pragma unroll
            for (int e = 0; e < EPL; ++e) lo[kg][rr][d0 + e] = o[rr][e];
        }
        __syncthreads();
        for (int idx = tid; idx < RC * D; idx += 256) {
            const int rr = idx / D, d = idx % D;
            const int r = r0 + rr;
            if (r >= R) continue;
            float M = -INFINITY;
            for (int k2 = 0; k2 < KGROUPS; ++k2) M = fmaxf(M, lm[k2][rr]);
            float O = 0.f, S = 0.f;
            for (int k2 = 0; k2 < KGROUPS; ++k2) {
                const float mk = lm[k2][rr];
                const float w = (mk == -INFINITY) ? 0.f : exp2f(mk - M);
                O += lo[k2][rr][d] * w;
                S += ll[k2][rr] * w;
            }
            const int i = r / gs, h = g * gs + (r % gs);
            const int m = rowbase + i;
            float* pp = a.part + (((size_t)m * Hq + h) * a.nsplit_max + split) * (D + 2);
            store_coherent(pp + 2 + d, O);
            if (d == 0) {
                store_coherent(pp, M);
                store_coherent(pp + 1, S);
            }
        }
        __syncthreads();
    }
}

// Merge of the split partials: one workgroup per (activation row, query head),
// one thread per output element; splits combined in split order.
template <int D>
__global__ __launch_bounds__(D) void attn_merge_kernel(AttnArgs a) {
    __shared__ float wgt[ATTN_MAX_SPLITS];
    __shared__ float inv_s;
    const int m = blockIdx.x, h = blockIdx.y, d = threadIdx.x;
    const ReqDev rq = a.meta.items[a.meta.row_item[m]].rq;    // the request of row m
    const int L = rq.P + rq.n;
    const int split_len = rq.split_len;
    const int nsplit = (L + split_len - 1) / split_len;
    const float* pp = a.part + ((size_t)m * a.Hq + h) * a.nsplit_max * (D + 2);
    if (d < 32) {
        float M = -INFINITY;
        for (int s2 = d; s2 < nsplit; s2 += 32) M = fmaxf(M, pp[(size_t)s2 * (D + 2)]);
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 32));
        float S = 0.f;
        for (int s2 = d; s2 < nsplit; s2 += 32) {
            const float ms = pp[(size_t)s2 * (D + 2)];
            const float w = (ms == -INFINITY) ? 0.f : exp2f(ms - M);
            wgt[s2] = w;
            S += pp[(size_t)s2 * (D + 2) + 1] * w;
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) S += __shfl_xor(S, o, 32);
        if (d == 0) inv_s = 1.0f / S;
    }
    __syncthreads();
    float O = 0.f;
    for (int s2 = 0; s2 < nsplit; ++s2) O += pp[(size_t)s2 * (D + 2) + 2 + d] * wgt[s2];
    a.out[(size_t)m * a.out_ld + (size_t)h * D + d] = O * inv_s;
    if (a.bp_out)                                            // the o product's input (64-row blocks)
        bp_put(a.bp_out + (size_t)(m >> 6) * 64 * a.kp, a.bc_out + (size_t)(m >> 6) * 2 * a.kp, a.kp, m & 63, h * D + d,
               O * inv_s, true);
}

// ------------------------------------------------------------------ matrix-core attention
//
// Same work split, partial format and append as attn_kernel, with the products
// on the matrix cores: every query vector of the (item, kv head) meets each
// 32-key step once.  Per 16-key subtile the scores are S^T = K Q^T (cache rows
// are the A operand as stored; q is split into a rounded part and its residual,
// both in the cache dtype, so the scores carry nearly fp32 precision), and the
// output is O^T += V^T P^T with P^T taken straight from the score registers
// (lane l holds keys 4 (l / 16) + j of both subtiles: exactly the k-slots of
// the B operand) and V^T read from a transposed copy of the value tile in LDS
// whose key slots follow the same order.  Keys a query may not see enter as
// zero rows with a -inf score.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
constexpr int AK = 32;                   // keys per step
constexpr int ACH = 512;                 // keys whose table entry and mask byte are staged at once

template <int KVDT>
__device__ __forceinline__ f32x4_t mma_kv(const u32x4& A, const u32x4& B, f32x4_t c) {
    if constexpr (KVDT == DT_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, A), __builtin_bit_cast(bf16x8_t, B), c,
                                                       0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, A), __builtin_bit_cast(half8_t, B), c, 0,
                                                      0, 0);
}
template <int KVDT>
__device__ __forceinline__ uint16_t kv_round(float f) { return KVDT == DT_BF16 ? f32_to_bf16(f) : f32_to_f16(f); }
template <int KVDT>
__device__ __forceinline__ float kv_float(uint16_t b) { return KVDT == DT_BF16 ? bf16_to_f32(b) : f16_to_f32(b); }
// Two floats rounded to the cache dtype (to nearest even) and packed, low half
// first: one v_cvt_pk_bf16_f32 for bf16.  Equal to kv_round of each for every
// finite input that is not an fp32 denormal (the probabilities it packs never are).
template <int KVDT>
__device__ __forceinline__ uint32_t kv_pack2(float lo, float hi) {
    if constexpr (KVDT == DT_BF16) {
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
        return __builtin_bit_cast(uint32_t, v);
    } else {
        return (uint32_t)kv_round<KVDT>(lo) | ((uint32_t)kv_round<KVDT>(hi) << 16);
    }
}

// The values of v in this lane and in lane ^ sh (sh = 16 or 32): every lane of
// the pair receives the lower lane's value in a and the upper lane's in b.
__device__ __forceinline__ void lane_pair_k(float v, int sh, float& a, float& b) {
    const uint32_t u = __float_as_uint(v);
    if (sh == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    }
}

// QTW: query tiles per wave per pass (which wave computes a query vector, and
// when, does not change its arithmetic).
template <int D, int KVDT, int QTW, bool REC = false>
__global__ __launch_bounds__(256, QTW == 1 ? 2 : 1) void attn_mma_kernel(AttnArgs a) {
    constexpr int HALF = D / 2;
    constexpr int NCH = D / 8;               // 16-byte chunks per cache row
    constexpr int DB = D / 32;               // k-blocks of the score products
    constexpr int MB = D / 16;               // row blocks of O^T
    constexpr int NU = AK * NCH / 256;       // chunks per thread per step (K and V each)
    constexpr int NS = ACH / 256;            // staged table entries per thread
    constexpr int VST = 40;                  // V^T row stride in elements (32 key slots + padding)
    static_assert(NU >= 1 && AK * NCH % 256 == 0, "tile staging");
    __shared__ __attribute__((aligned(16))) uint16_t ks[2][AK][D];   // key rows, chunk c at c ^ (key mod NCH)
    __shared__ __attribute__((aligned(16))) uint16_t vt[2][D][VST];  // values transposed, key slots permuted
    __shared__ int16_t stab[ACH];                                    // physical slot of each key of the chunk
    __shared__ __attribute__((aligned(16))) uint8_t smk[ACH];        // its mask byte (read as words)

    const int item = blockIdx.x, g = blockIdx.y, split = blockIdx.z;
    const ItemDev it = a.meta.items[item];
    const ReqDev rq = it.rq;
    const int b = it.slot;
    const int P = rq.P, n = rq.n;
    const int L = P + n;
    const int split_len = rq.split_len;
    const int nsplit = (L + split_len - 1) / split_len;
    if (split >= nsplit) return;
    const int j0 = split * split_len, j1 = min(L, j0 + split_len);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ql = lane & 15, lg = lane >> 4;
    const int Hq = a.Hq, Hkv = a.Hkv;
    const int gs = Hq / Hkv;
    const int R = gs * n;
    const int nqt = (R + 15) / 16;
    const size_t lstride = (size_t)rq.S * Hkv * rq.cap * D;
    uint16_t* kl = rq.kc + (size_t)a.layer * lstride;
    uint16_t* vl = rq.vc + (size_t)a.layer * lstride;
    const uint8_t* mask = a.meta.masks + rq.mask_off + (size_t)b * rq.mask_len;
    // per-query-row masks of the slot, [n][mask_len], when the request has them
    const uint8_t* rmask = rq.rowmask_off >= 0 ? a.meta.masks + rq.rowmask_off + (size_t)b * n * rq.mask_len : nullptr;
    const int16_t* tab = rq.table + (size_t)b * rq.cap;
    const int rowbase = rq.row0 + b * n;

    // ---- one step's keys (chunk-relative key x0 + k): cache rows through the
    // table, this forward's rows from q|k|v.  Cache rows are loaded without
    // branches (clamped to an allocated row; whether a chunk is kept is a bit
    // applied when it is staged), so the mask and table reads are all in flight
    // at once and nothing waits for the loads before the staging.
    u32x4 kreg[NU], vreg[NU];
    uint32_t keep = 0u;
    int c0 = j0, c1 = j0;                                    // keys of the staged chunk
    auto fetch = [&](int x0, bool append) {
        uint32_t kb_ = 0u;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int q = tid + 256 * u, k = q / NCH, c = q % NCH;
            const int x = min(x0 + k, ACH - 1), j = c0 + x0 + k;
            const bool cached = j < min(c1, P);
            const int slot = cached ? (int)stab[x] : b;
            const size_t off = (((size_t)slot * Hkv + g) * rq.cap + (cached ? j : 0)) * D + 8 * c;
            kreg[u] = *(const u32x4*)(kl + off);
            vreg[u] = *(const u32x4*)(vl + off);
            kb_ |= ((cached && smk[x] != 0) ? 1u : 0u) << u;
        }
        if (c0 + x0 + AK > P && c0 + x0 < c1) {              // the step holds rows of this forward (uniform)
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int q = tid + 256 * u, k = q / NCH, c = q % NCH;
                const int x = min(x0 + k, ACH - 1), j = c0 + x0 + k;
                if (j < P || j >= c1) continue;
                const int i = j - P;
                const int m = rowbase + i;
                const int pos = a.meta.positions[m];
                const float* krow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + g) * D;
                const float* vrow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + Hkv + g) * D;
                uint16_t kb[8], vb[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int d = 8 * c + e;
                    const bool lo_half = d < HALF;
                    const float xk = krow[d];
                    const float xp = lo_half ? krow[d + HALF] : krow[d - HALF];
                    const float2 cs = a.rope[(size_t)pos * HALF + (lo_half ? d : d - HALF)];
                    const float y = lo_half ? (xk * cs.x - xp * cs.y) : (xk * cs.x + xp * cs.y);
                    kb[e] = kv_round<KVDT>(y);
                    vb[e] = kv_round<KVDT>(vrow[d]);
                }
                u32x4 kk, vv;
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2) {
                    kk[w2] = (uint32_t)kb[2 * w2] | ((uint32_t)kb[2 * w2 + 1] << 16);
                    vv[w2] = (uint32_t)vb[2 * w2] | ((uint32_t)vb[2 * w2 + 1] << 16);
                }
                if (append) {                                // append: owner of row j writes it
                    const size_t off = (((size_t)b * Hkv + g) * rq.cap + j) * D + 8 * c;
                    *(u32x4*)(kl + off) = kk;
                    *(u32x4*)(vl + off) = vv;
                    if (a.layer == 0 && g == 0 && c == 0) rq.table[(size_t)b * rq.cap + j] = (int16_t)b;
                }
                kreg[u] = kk;
                vreg[u] = vv;
                kb_ |= (smk[x] != 0 ? 1u : 0u) << u;
            }
        }
        keep = kb_;
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int q = tid + 256 * u, k = q / NCH, c = q % NCH;
            const bool kp_ = (keep >> u) & 1u;               // dropped chunks enter as zero rows
            const u32x4 kv = kreg[u], vv = vreg[u];
            *(u32x4*)&ks[buf][k][8 * (c ^ (k % NCH))] = u32x4{kp_ ? kv[0] : 0u, kp_ ? kv[1] : 0u, kp_ ? kv[2] : 0u, kp_ ? kv[3] : 0u};
            const int slot = 8 * ((k & 15) >> 2) + 4 * (k >> 4) + (k & 3);
#pragma unroll
            for (int e = 0; e < 8; ++e) vt[buf][8 * c + e][slot] = kp_ ? (uint16_t)(vv[e >> 1] >> (16 * (e & 1))) : (uint16_t)0;
        }
    };

    // table entries and mask bytes of the first chunk
    int16_t ptab[NS];
    uint8_t pmsk[NS];
#pragma unroll
    for (int t2 = 0; t2 < NS; ++t2) {
        const int j = j0 + tid + 256 * t2;
        const bool in = j < min(j1, j0 + ACH);
        pmsk[t2] = in ? mask[j] : 0;
        ptab[t2] = (in && j < P) ? tab[j] : (int16_t)b;
    }
    // ---- the first chunk's mask bytes and table entries are staged and its first
    // step's loads issued before the queries are set up: they fly during it
    c1 = min(j1, j0 + ACH);
#pragma unroll
    for (int t2 = 0; t2 < NS; ++t2) {
        smk[tid + 256 * t2] = pmsk[t2];
        stab[tid + 256 * t2] = ptab[t2];
    }
    __syncthreads();
    fetch(0, !a.no_append);
    for (int qg = 0; qg < nqt; qg += 4 * QTW) {
        // ---- this wave's query tiles: rotated, scaled, split into rounded part and residual
        u32x4 qh[QTW][DB], qr[QTW][DB];
        int qtok[QTW];
        float mrun[QTW], lsum[QTW];
        f32x4_t o[QTW][MB];
#pragma unroll
        for (int u = 0; u < QTW; ++u) {
            const int qt = qg + wave + 4 * u;
            const int r = 16 * qt + ql;
            const bool ok = qt < nqt && r < R;
            const int i = ok ? r / gs : 0, h = g * gs + (ok ? r % gs : 0);
            const int m = rowbase + i;
            const float* qrow = a.qkv + (size_t)m * a.qkv_ld + (size_t)h * D;
            qtok[u] = ok ? i : n;
            // every load of the tile at once (row 0 of the item stands in for a missing
            // row): q and its rotary partners, then (cos, sin) at the row's position
            float4 qa[DB][2], qp[DB][2], rc[DB][4];
#pragma unroll
            for (int ib = 0; ib < DB; ++ib) {
                const int d0 = 32 * ib + 8 * lg;
                const bool lo_half = d0 < HALF;
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    qa[ib][h2] = ((const float4*)(qrow + d0))[h2];
                    qp[ib][h2] = ((const float4*)(qrow + (lo_half ? d0 + HALF : d0 - HALF)))[h2];
                }
            }
            const int pos = a.meta.positions[m];
#pragma unroll
            for (int ib = 0; ib < DB; ++ib) {
                const int d0 = 32 * ib + 8 * lg;
                const float4* r4 = (const float4*)(a.rope + (size_t)pos * HALF + (d0 < HALF ? d0 : d0 - HALF));
#pragma unroll
                for (int h4 = 0; h4 < 4; ++h4) rc[ib][h4] = r4[h4];
            }
#pragma unroll
            for (int ib = 0; ib < DB; ++ib) {
                // dims d0 .. d0 + 7 lie in one rotary half
                const int d0 = 32 * ib + 8 * lg;
                const bool lo_half = d0 < HALF;
                float xv[8], xpv[8], cv[8], sv[8];
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    const float4 x4 = qa[ib][h2], y4 = qp[ib][h2];
                    xv[4 * h2] = x4.x; xv[4 * h2 + 1] = x4.y; xv[4 * h2 + 2] = x4.z; xv[4 * h2 + 3] = x4.w;
                    xpv[4 * h2] = y4.x; xpv[4 * h2 + 1] = y4.y; xpv[4 * h2 + 2] = y4.z; xpv[4 * h2 + 3] = y4.w;
                }
#pragma unroll
                for (int h4 = 0; h4 < 4; ++h4) {
                    const float4 c4 = rc[ib][h4];
                    cv[2 * h4] = c4.x; sv[2 * h4] = c4.y; cv[2 * h4 + 1] = c4.z; sv[2 * h4 + 1] = c4.w;
                }
                uint16_t hb[8], rb[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float y = 0.f;
                    if (ok) y = lo_half ? (xv[e] * cv[e] - xpv[e] * sv[e]) : (xv[e] * cv[e] + xpv[e] * sv[e]);
                    if constexpr (REC) if (ok) a.dbg_q[((size_t)m * Hq + h) * D + d0 + e] = y;
                    y *= a.qscale;
                    hb[e] = kv_round<KVDT>(y);
                    rb[e] = kv_round<KVDT>(y - kv_float<KVDT>(hb[e]));
                }
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2) {
                    qh[u][ib][w2] = (uint32_t)hb[2 * w2] | ((uint32_t)hb[2 * w2 + 1] << 16);
                    qr[u][ib][w2] = (uint32_t)rb[2 * w2] | ((uint32_t)rb[2 * w2 + 1] << 16);
                }
            }
            mrun[u] = -INFINITY;
            lsum[u] = 0.f;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) o[u][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }

        for (c0 = j0; c0 < j1; c0 += ACH) {
        c1 = min(j1, c0 + ACH);
        if (qg != 0 || c0 != j0) {                           // (the first chunk was staged above)
            __syncthreads();                                 // the previous chunk's entries are no longer read
            for (int x = tid; x < c1 - c0; x += 256) {
                const int j = c0 + x;
                smk[x] = mask[j];
                stab[x] = j < P ? tab[j] : (int16_t)b;
            }
            __syncthreads();
            fetch(0, qg == 0 && !a.no_append);
        }
        const int nsteps = (c1 - c0 + AK - 1) / AK;
        stash(0);
        __syncthreads();
        for (int st = 0; st < nsteps; ++st) {
            const int buf = st & 1;
            if (st + 1 < nsteps) fetch((st + 1) * AK, qg == 0 && !a.no_append);   // next step's loads fly during this one
            // the lane's 8 keys: step key 4 lg + e (e < 4) or 16 + 4 lg + e - 4; visible ones as bits
            const int kbase = c0 + st * AK + 4 * lg;
            uint32_t vbits = 0u;
            {
                // mask bytes of keys 4 lg + 0..3 and 16 + 4 lg + 0..3 as two aligned words
                const uint32_t w0 = *(const uint32_t*)&smk[st * AK + 4 * lg];
                const uint32_t w1 = *(const uint32_t*)&smk[st * AK + 16 + 4 * lg];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int ko = (e < 4) ? e : 12 + e;
                    const uint32_t byte = ((e < 4 ? w0 : w1) >> (8 * (e & 3))) & 0xFFu;
                    vbits |= ((kbase + ko < c1 && byte != 0u) ? 1u : 0u) << e;
                }
            }
#pragma unroll
            for (int u = 0; u < QTW; ++u) {
                if (qg + wave + 4 * u >= nqt) continue;      // wave-uniform
                f32x4_t s0 = f32x4_t{0.f, 0.f, 0.f, 0.f}, s1 = s0;
                u32x4 kf0[DB], kf1[DB];                      // every key fragment of the step in flight at once
#pragma unroll
                for (int ib = 0; ib < DB; ++ib) {
                    const int c = 4 * ib + lg;
                    kf0[ib] = *(const u32x4*)&ks[buf][ql][8 * (c ^ (ql % NCH))];
                    kf1[ib] = *(const u32x4*)&ks[buf][16 + ql][8 * (c ^ ((16 + ql) % NCH))];
                }
#pragma unroll
                for (int ib = 0; ib < DB; ++ib) {
                    s0 = mma_kv<KVDT>(kf0[ib], qh[u][ib], s0);
                    s1 = mma_kv<KVDT>(kf1[ib], qh[u][ib], s1);
                    s0 = mma_kv<KVDT>(kf0[ib], qr[u][ib], s0);
                    s1 = mma_kv<KVDT>(kf1[ib], qr[u][ib], s1);
                }
                u32x4 vf[MB];                                // value fragments: read during the softmax
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) vf[mb] = *(const u32x4*)&vt[buf][16 * mb + ql][8 * lg];
                const int last = P + qtok[u] - kbase;         // keys up to kbase + last are causal
                float sv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int ko = (e < 4) ? e : 12 + e;
                    const float x = e < 4 ? s0[e] : s1[e - 4];
                    sv[e] = (((vbits >> e) & 1u) && ko <= last) ? x : -INFINITY;
                }
                if (rmask) {                                 // this query row's own mask (uniform branch)
                    const uint8_t* rrow = rmask + (size_t)min(qtok[u], n - 1) * rq.mask_len;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int j = min(kbase + ((e < 4) ? e : 12 + e), rq.mask_len - 1);
                        if (rrow[j] == 0) sv[e] = -INFINITY;
                    }
                }
                if constexpr (REC) {                             // test support: this tile's visible scores
                    const int r = 16 * (qg + wave + 4 * u) + ql;
                    if (r < R) {
                        const size_t row = ((size_t)(rowbase + r / gs) * Hq + g * gs + r % gs) * a.dbg_keys;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int j = kbase + ((e < 4) ? e : 12 + e);
                            if (sv[e] != -INFINITY && j < a.dbg_keys) a.dbg_logits[row + j] = sv[e] * 0.69314718055994531f;
                        }
                    }
                }
                float mx = sv[0];
#pragma unroll
                for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
                float x0, x1;
                lane_pair_k(mx, 16, x0, x1);
                mx = fmaxf(x0, x1);
                lane_pair_k(mx, 32, x0, x1);
                mx = fmaxf(x0, x1);
                const float mn = fmaxf(mrun[u], mx);
                // no key seen yet (mn = -inf): base 0 makes every term and the correction 0
                const float base = mn == -INFINITY ? 0.f : mn;
                const float corr = __builtin_amdgcn_exp2f(mrun[u] - base);
                float pv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(sv[e] - base);
                float ps = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) ps += pv[e];
                lsum[u] = lsum[u] * corr + ps;
                mrun[u] = mn;
                u32x4 pb;
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2) pb[w2] = kv_pack2<KVDT>(pv[2 * w2], pv[2 * w2 + 1]);
                if (__any(corr != 1.f)) {                        // the running maximum moved in some lane
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj) o[u][mb][jj] *= corr;
                }
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) o[u][mb] = mma_kv<KVDT>(vf[mb], pb, o[u][mb]);
            }
            if (st + 1 < nsteps) stash(buf ^ 1);
            __syncthreads();
        }
        }

        // ---- this split's partial of each query vector: (max, sum, unnormalized output)
#pragma unroll
        for (int u = 0; u < QTW; ++u) {
            const int qt = qg + wave + 4 * u;
            if (qt >= nqt) continue;
            float x0, x1, lt = lsum[u];
            lane_pair_k(lt, 16, x0, x1);
            lt = x0 + x1;
            lane_pair_k(lt, 32, x0, x1);
            lt = x0 + x1;
            const int r = 16 * qt + ql;
            if (r >= R) continue;
            const int i = r / gs, h = g * gs + (r % gs);
            const int m = rowbase + i;
            float* pp = a.part + (((size_t)m * Hq + h) * a.nsplit_max + split) * (D + 2);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) pp[2 + 16 * mb + 4 * lg + jj] = o[u][mb][jj];
            if (lg == 0) {
                pp[0] = mrun[u];
                pp[1] = lt;
            }
        }
    }
}

// ------------------------------------------------------------------ matrix-core attention, cache rows by direct loads
//
// attn_mma_kernel for items of at most 256 query vectors per kv head (up to four
// tiles per wave), with the same split, step order, arithmetic and partials
// (results are bitwise equal), but with the cache rows of each 32-key step
// brought into LDS by direct-to-LDS buffer loads issued ATTN_NB - 1 steps ahead
// instead of through registers one step ahead.  A key the split does not keep (masked,
// past the split, or a row of this forward, which is written in afterwards)
// is read at an offset past the buffer's end, which the hardware answers with
// zeros without a memory access.  K and V are stored as in memory, 16-byte
// chunk c of key k at position c ^ (k mod chunks per row); the value fragments
// of O^T += V^T P^T come from ds_read_b64_tr_b16, which hands lane i of each
// 16-lane group element i mod 4 of the 8 bytes read by lane 4 e + i / 4 of the
// group, as element e (e < 4): the four keys of a fragment half become one
// lane's four k slots.  The whole split's table entries and mask bytes (at
// most ATTN_SCH keys) and the rows of a per-query-row mask (at most ATTN_RSM
// bytes) are staged first; LDS is read through inline assembly and the
// workgroup synchronizes with a bare s_barrier, so no compiler-inserted wait
// drains the loads in flight.
constexpr int ATTN_NB = 4;                // step buffers (K and V of 32 keys each)
constexpr int ATTN_SCH = 1024;            // most keys of one split on this path
constexpr int ATTN_RSM = 8192;            // bytes of per-query-row mask staged per split (rows x split keys)

__device__ __forceinline__ void attn_dma(__amdgpu_buffer_rsrc_t r, uint32_t off, void* lds) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, off, 0, 0, 2 /* nt */);
}
__device__ __forceinline__ u32x4 attn_lds16(uint32_t a) {
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(a));
    return v;
}
__device__ __forceinline__ u32x2 attn_lds_tr(uint32_t a) {
    u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(v) : "v"(a));
    return v;
}
__device__ __forceinline__ uint32_t attn_lds4(uint32_t a) {
    uint32_t v;
    asm volatile("ds_read_b32 %0, %1" : "=v"(v) : "v"(a));
    return v;
}
__device__ __forceinline__ uint32_t attn_lds_u16(uint32_t a) {
    uint32_t v;
    asm volatile("ds_read_u16 %0, %1" : "=v"(v) : "v"(a));
    return v;
}
__device__ __forceinline__ uint32_t attn_lds_u8(uint32_t a) {
    uint32_t v;
    asm volatile("ds_read_u8 %0, %1" : "=v"(v) : "v"(a));
    return v;
}
__device__ __forceinline__ void attn_lgkm() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// After attn_lgkm: makes v depend on the wait, so no use of a value read by
// inline assembly moves above it (the compiler takes such values as ready).
__device__ __forceinline__ void touch_v(u32x4& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void touch_u(uint32_t& v) { asm volatile("" : "+v"(v)); }
template <int N>
__device__ __forceinline__ void attn_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void attn_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A workgroup takes 64 query vectors of one (item, kv head) and one split of its
// keys, a tile of 16 per wave; items with more are spread over blockIdx.z.  The
// workgroups of one split's query blocks are items x kv heads x nsplit_max apart,
// so they read the same rows on the same XCD where that is a multiple of 8 (8 kv
// heads: always).  (Several tiles per wave spilled registers and left most CUs
// without work: 64 rows at KV 2048 were 72 workgroups, 60 us.)
template <int D, int KVDT, bool REC = false>
__global__ __launch_bounds__(256, 2) void attn_dma_kernel(AttnArgs a) {
    constexpr int HALF = D / 2;
    constexpr int NCH = D / 8;               // 16-byte chunks per cache row
    constexpr int DB = D / 32;               // k-blocks of the score products
    constexpr int MB = D / 16;               // row blocks of O^T
    constexpr int RB = 2 * D;                // bytes per cache row
    constexpr int SB = AK * RB;              // bytes of one step's K (or V)
    constexpr int KPI = 1024 / RB;           // keys per direct load (64 lanes x 16 bytes)
    constexpr int NI = SB / 1024 / 4;        // direct loads per wave per step, K and V each
    constexpr int VMN = 2 * NI * (ATTN_NB - 2);   // loads a lane may leave in flight at the top of a step
    static_assert(NI >= 1 && VMN <= 63, "step geometry");
    static_assert(AK * NCH % 256 == 0, "new-row staging");
    __shared__ __attribute__((aligned(16))) uint8_t kvs[ATTN_NB][2][SB];
    __shared__ int16_t stab[ATTN_SCH];
    __shared__ __attribute__((aligned(16))) uint8_t smk[ATTN_SCH];
    __shared__ __attribute__((aligned(16))) uint8_t srm[ATTN_RSM];   // [row][split key] when the request has row masks

    const int item = blockIdx.x, g = blockIdx.y, split = blockIdx.z % a.nsplit_max, qb = blockIdx.z / a.nsplit_max;
    const ItemDev it = a.meta.items[item];
    const ReqDev rq = it.rq;
    const int b = it.slot;
    const int P = rq.P, n = rq.n;
    const int L = P + n;
    const int split_len = rq.split_len;
    const int nsplit = (L + split_len - 1) / split_len;
    if (split >= nsplit) return;
    const int j0 = split * split_len, j1 = min(L, j0 + split_len);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ql = lane & 15, lg = lane >> 4;
    const int Hq = a.Hq, Hkv = a.Hkv;
    const int gs = Hq / Hkv;
    const int R = gs * n;
    if (64 * qb >= R) return;                                // whole workgroup
    const size_t lstride = (size_t)rq.S * Hkv * rq.cap * D;
    uint16_t* kl = rq.kc + (size_t)a.layer * lstride;
    uint16_t* vl = rq.vc + (size_t)a.layer * lstride;
    const uint8_t* mask = a.meta.masks + rq.mask_off + (size_t)b * rq.mask_len;
    const int16_t* tab = rq.table + (size_t)b * rq.cap;
    const int rowbase = rq.row0 + b * n;

    // ---- the split's table entries and mask bytes (and each query row's own mask)
    for (int x = tid; x < j1 - j0; x += 256) {
        const int j = j0 + x;
        smk[x] = mask[j];
        stab[x] = j < P ? tab[j] : (int16_t)b;
    }
    const uint8_t* rmask = rq.rowmask_off >= 0 ? a.meta.masks + rq.rowmask_off + (size_t)b * n * rq.mask_len : nullptr;
    const int rspan = (j1 - j0 + 3) & ~3;                    // row stride of srm (the host checked n * rspan fits)
    if (rmask)
        for (int q = tid; q < n * rspan; q += 256) {
            const int i = q / rspan, x = q - i * rspan;
            srm[q] = x < j1 - j0 ? rmask[(size_t)i * rq.mask_len + j0 + x] : (uint8_t)0;
        }
    __syncthreads();

    // ---- direct loads of step s into buffer s mod ATTN_NB: lane l of load h of
    // this wave carries chunk position l mod NCH of key (NI wave + h) KPI + l / NCH
    const int nsteps = (j1 - j0 + AK - 1) / AK;
    const uint32_t lbytes = (uint32_t)(lstride * 2);
    const __amdgpu_buffer_rsrc_t rk = buf_rsrc(kl, lbytes), rv = buf_rsrc(vl, lbytes);
    const uint32_t smk_a = (uint32_t)(uintptr_t)smk, stab_a = (uint32_t)(uintptr_t)stab;
    const uint32_t kvs_a = (uint32_t)(uintptr_t)&kvs[0][0][0];
    const int cstop = min(j1, P);                            // keys below this come from the cache
    auto issue = [&](int s) {
        uint32_t off[NI];
#pragma unroll
        for (int h = 0; h < NI; ++h) {
            const int key = (NI * wave + h) * KPI + lane / NCH;
            const int x = min(s * AK + key, ATTN_SCH - 1), j = j0 + s * AK + key;
            uint32_t mk = attn_lds_u8(smk_a + (uint32_t)x);
            uint32_t tb = attn_lds_u16(stab_a + 2u * (uint32_t)x);
            attn_lgkm();
            touch_u(mk);
            touch_u(tb);
            const int slot = (int)(int16_t)tb;
            const int c = (lane % NCH) ^ (key % NCH);
            const bool kept = s < nsteps && j < cstop && mk != 0u;
            off[h] = kept ? (uint32_t)(((((size_t)slot * Hkv + g) * rq.cap + j) * D + 8 * c) * 2) : 0xFFFFFFF0u;
        }
        uint8_t* kb = &kvs[s % ATTN_NB][0][0];
#pragma unroll
        for (int h = 0; h < NI; ++h) {
            const int blk = (NI * wave + h) * 1024;
            attn_dma(rk, off[h], kb + blk);
            attn_dma(rv, off[h], kb + SB + blk);
        }
    };
#pragma unroll
    for (int s = 0; s < ATTN_NB - 1; ++s) issue(s);

    // ---- this wave's query tiles: rotated, scaled, split into rounded part and residual
    const int r = 64 * qb + 16 * wave + ql;                  // this lane's query vector
    const bool active = 64 * qb + 16 * wave < R;
    u32x4 qh[DB], qr[DB];
    int qtok;
    float mrun, lsum;
    f32x4_t o[MB];
    {
        const bool ok = r < R;
        const int i = ok ? r / gs : 0, h = g * gs + (ok ? r % gs : 0);
        const int m = rowbase + i;
        const float* qrow = a.qkv + (size_t)m * a.qkv_ld + (size_t)h * D;
        qtok = ok ? i : n;
        mrun = -INFINITY;
        lsum = 0.f;
        // every load of the tile at once (row 0 of the item stands in for a missing
        // row): q and its rotary partners, then (cos, sin) at the row's position
        float4 qa[DB][2], qp[DB][2], rc[DB][4];
#pragma unroll
        for (int ib = 0; ib < DB; ++ib) {
            const int d0 = 32 * ib + 8 * lg;
            const bool lo_half = d0 < HALF;
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                qa[ib][h2] = ((const float4*)(qrow + d0))[h2];
                qp[ib][h2] = ((const float4*)(qrow + (lo_half ? d0 + HALF : d0 - HALF)))[h2];
            }
        }
        const int pos = a.meta.positions[m];
#pragma unroll
        for (int ib = 0; ib < DB; ++ib) {
            const int d0 = 32 * ib + 8 * lg;
            const float4* r4 = (const float4*)(a.rope + (size_t)pos * HALF + (d0 < HALF ? d0 : d0 - HALF));
#pragma unroll
            for (int h4 = 0; h4 < 4; ++h4) rc[ib][h4] = r4[h4];
        }
#pragma unroll
        for (int ib = 0; ib < DB; ++ib) {
            // dims d0 .. d0 + 7 lie in one rotary half
            const int d0 = 32 * ib + 8 * lg;
            const bool lo_half = d0 < HALF;
            float xv[8], xpv[8], cv[8], sv[8];
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const float4 x4 = qa[ib][h2], y4 = qp[ib][h2];
                xv[4 * h2] = x4.x; xv[4 * h2 + 1] = x4.y; xv[4 * h2 + 2] = x4.z; xv[4 * h2 + 3] = x4.w;
                xpv[4 * h2] = y4.x; xpv[4 * h2 + 1] = y4.y; xpv[4 * h2 + 2] = y4.z; xpv[4 * h2 + 3] = y4.w;
            }
#pragma unroll
            for (int h4 = 0; h4 < 4; ++h4) {
                const float4 c4 = rc[ib][h4];
                cv[2 * h4] = c4.x; sv[2 * h4] = c4.y; cv[2 * h4 + 1] = c4.z; sv[2 * h4 + 1] = c4.w;
            }
            uint16_t hb[8], rb[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float y = 0.f;
                if (ok) y = lo_half ? (xv[e] * cv[e] - xpv[e] * sv[e]) : (xv[e] * cv[e] + xpv[e] * sv[e]);
                if constexpr (REC) if (ok) a.dbg_q[((size_t)m * Hq + h) * D + d0 + e] = y;
                y *= a.qscale;
                hb[e] = kv_round<KVDT>(y);
                rb[e] = kv_round<KVDT>(y - kv_float<KVDT>(hb[e]));
            }
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) {
                qh[ib][w2] = (uint32_t)hb[2 * w2] | ((uint32_t)hb[2 * w2 + 1] << 16);
                qr[ib][w2] = (uint32_t)rb[2 * w2] | ((uint32_t)rb[2 * w2 + 1] << 16);
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) o[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    for (int st = 0; st < nsteps; ++st) {
        const int buf = st % ATTN_NB;
        if constexpr (REC) attn_vm<0>();                     // the record's stores share the load counter
        else attn_vm<VMN>();                                 // this step's loads (later steps may stay in flight)
        attn_barrier();                                      // every lane's loads of this step are in LDS
        issue(st + ATTN_NB - 1);                             // into the buffer every wave finished with
        const int x0 = st * AK;
        if (j0 + x0 + AK > P && j0 + x0 < j1) {              // the step holds rows of this forward (uniform)
            uint8_t* kb = &kvs[buf][0][0];
#pragma unroll
            for (int u = 0; u < AK * NCH / 256; ++u) {
                const int q = tid + 256 * u, k = q / NCH, c = q % NCH;
                const int j = j0 + x0 + k;
                if (j < P || j >= j1) continue;
                const int i = j - P;
                const int m = rowbase + i;
                const int pos = a.meta.positions[m];
                const float* krow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + g) * D;
                const float* vrow = a.qkv + (size_t)m * a.qkv_ld + (size_t)(Hq + Hkv + g) * D;
                uint16_t kb8[8], vb8[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int d = 8 * c + e;
                    const bool lo_half = d < HALF;
                    const float xk = krow[d];
                    const float xp = lo_half ? krow[d + HALF] : krow[d - HALF];
                    const float2 cs = a.rope[(size_t)pos * HALF + (lo_half ? d : d - HALF)];
                    const float y = lo_half ? (xk * cs.x - xp * cs.y) : (xk * cs.x + xp * cs.y);
                    kb8[e] = kv_round<KVDT>(y);
                    vb8[e] = kv_round<KVDT>(vrow[d]);
                }
                u32x4 kk, vv;
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2) {
                    kk[w2] = (uint32_t)kb8[2 * w2] | ((uint32_t)kb8[2 * w2 + 1] << 16);
                    vv[w2] = (uint32_t)vb8[2 * w2] | ((uint32_t)vb8[2 * w2 + 1] << 16);
                }
                if (qb == 0) {                               // append: owner of row j writes it
                    const size_t off = (((size_t)b * Hkv + g) * rq.cap + j) * D + 8 * c;
                    *(u32x4*)(kl + off) = kk;
                    *(u32x4*)(vl + off) = vv;
                    if (a.layer == 0 && g == 0 && c == 0) rq.table[(size_t)b * rq.cap + j] = (int16_t)b;
                }
                if (smk[x0 + k] != 0) {                      // a kept row enters; a dropped one stays zero
                    const int pos16 = 16 * (c ^ (k % NCH));
                    *(u32x4*)(kb + k * RB + pos16) = kk;
                    *(u32x4*)(kb + SB + k * RB + pos16) = vv;
                }
            }
            attn_barrier();
        }
        if (active) {
            const uint32_t kb_a = kvs_a + (uint32_t)(buf * 2 * SB), vb_a = kb_a + SB;
            const int kbase = j0 + x0 + 4 * lg;
            u32x4 kf0[DB], kf1[DB], vf[MB];
#pragma unroll
            for (int ib = 0; ib < DB; ++ib) {
                const int c = 4 * ib + lg;
                kf0[ib] = attn_lds16(kb_a + (uint32_t)(ql * RB + 16 * (c ^ (ql % NCH))));
                kf1[ib] = attn_lds16(kb_a + (uint32_t)((16 + ql) * RB + 16 * (c ^ ((16 + ql) % NCH))));
            }
            // value fragments: read h gives keys 16 h + 4 lg + e; this lane supplies
            // key 16 h + 4 lg + ql / 4, dims 16 mb + 4 (ql mod 4) .. + 3
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                u32x2 p0, p1;
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int key = 16 * hh + 4 * lg + (ql >> 2);
                    const int d = 16 * mb + 4 * (ql & 3);
                    const uint32_t ad = vb_a + (uint32_t)(key * RB + 16 * ((d >> 3) ^ (key % NCH)) + 2 * (d & 7));
                    if (hh == 0) p0 = attn_lds_tr(ad);
                    else p1 = attn_lds_tr(ad);
                }
                vf[mb] = u32x4{p0[0], p0[1], p1[0], p1[1]};
            }
            uint32_t w0 = attn_lds4(smk_a + (uint32_t)(x0 + 4 * lg));
            uint32_t w1 = attn_lds4(smk_a + (uint32_t)(x0 + 16 + 4 * lg));
            attn_lgkm();
            touch_u(w0);
            touch_u(w1);
#pragma unroll
            for (int ib = 0; ib < DB; ++ib) { touch_v(kf0[ib]); touch_v(kf1[ib]); }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) touch_v(vf[mb]);
            uint32_t vb0 = 0u;                               // keys of the step this split keeps
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int ko = (e < 4) ? e : 12 + e;
                const uint32_t byte = ((e < 4 ? w0 : w1) >> (8 * (e & 3))) & 0xFFu;
                vb0 |= ((kbase + ko < j1 && byte != 0u) ? 1u : 0u) << e;
            }
            {
                uint32_t vbits = vb0;
                if (rmask) {                                 // this query row's own mask bytes (uniform branch)
                    const uint32_t ra = (uint32_t)(uintptr_t)srm + (uint32_t)(min(qtok, n - 1) * rspan + x0 + 4 * lg);
                    uint32_t r0 = attn_lds4(ra), r1 = attn_lds4(ra + 16);
                    attn_lgkm();
                    touch_u(r0);
                    touch_u(r1);
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if ((((e < 4 ? r0 : r1) >> (8 * (e & 3))) & 0xFFu) == 0u) vbits &= ~(1u << e);
                }
                f32x4_t s0 = f32x4_t{0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
                for (int ib = 0; ib < DB; ++ib) {
                    s0 = mma_kv<KVDT>(kf0[ib], qh[ib], s0);
                    s1 = mma_kv<KVDT>(kf1[ib], qh[ib], s1);
                    s0 = mma_kv<KVDT>(kf0[ib], qr[ib], s0);
                    s1 = mma_kv<KVDT>(kf1[ib], qr[ib], s1);
                }
                const int last = P + qtok - kbase;        // keys up to kbase + last are causal
                float sv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int ko = (e < 4) ? e : 12 + e;
                    const float x = e < 4 ? s0[e] : s1[e - 4];
                    sv[e] = (((vbits >> e) & 1u) && ko <= last) ? x : -INFINITY;
                }
                if constexpr (REC) {                         // test support: this tile's visible scores
                    if (r < R) {
                        const size_t row = ((size_t)(rowbase + r / gs) * Hq + g * gs + r % gs) * a.dbg_keys;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int j = kbase + ((e < 4) ? e : 12 + e);
                            if (sv[e] != -INFINITY && j < a.dbg_keys) a.dbg_logits[row + j] = sv[e] * 0.69314718055994531f;
                        }
                    }
                }
                float mx = sv[0];
#pragma unroll
                for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
                float x0f, x1f;
                lane_pair_k(mx, 16, x0f, x1f);
                mx = fmaxf(x0f, x1f);
                lane_pair_k(mx, 32, x0f, x1f);
                mx = fmaxf(x0f, x1f);
                const float mn = fmaxf(mrun, mx);
                // no key seen yet (mn = -inf): base 0 makes every term and the correction 0
                const float base = mn == -INFINITY ? 0.f : mn;
                const float corr = __builtin_amdgcn_exp2f(mrun - base);
                float pv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(sv[e] - base);
                float ps = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) ps += pv[e];
                lsum = lsum * corr + ps;
                mrun = mn;
                u32x4 pb;
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2) pb[w2] = kv_pack2<KVDT>(pv[2 * w2], pv[2 * w2 + 1]);
                if (__any(corr != 1.f)) {                    // the running maximum moved in some lane
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj) o[mb][jj] *= corr;
                }
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) o[mb] = mma_kv<KVDT>(vf[mb], pb, o[mb]);
            }
        }
    }
    attn_vm<0>();                                            // no direct load may land after the workgroup ends

    // ---- this split's partial of each query vector: (max, sum, unnormalized output)
    if (active) {
        float x0f, x1f, lt = lsum;
        lane_pair_k(lt, 16, x0f, x1f);
        lt = x0f + x1f;
        lane_pair_k(lt, 32, x0f, x1f);
        lt = x0f + x1f;
        if (r < R) {
            const int i = r / gs, h = g * gs + (r % gs);
            const int m = rowbase + i;
            float* pp = a.part + (((size_t)m * Hq + h) * a.nsplit_max + split) * (D + 2);
            // 16-byte stores (the record is only 8-byte aligned; the hardware takes
            // 4-byte aligned wide stores): a store per value lengthens the launch's drain
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) __builtin_memcpy(pp + 2 + 16 * mb + 4 * lg, &o[mb], 16);
            if (lg == 0) {
                const float2 ml = {mrun, lt};
                __builtin_memcpy(pp, &ml, 8);
            }
        }
    }
}

hipError_t launch_attention(const AttnArgs& a, int head_dim, int queries_per_item_max, hipStream_t st) {
    const dim3 grid(a.meta.n_items, a.Hkv, a.nsplit_max), block(256);
    const dim3 mgrid(a.meta.M, a.Hq);
    const bool wide = queries_per_item_max > 4;
    const bool bf = a.kv_dt == DT_BF16;
    const bool one = queries_per_item_max <= 64;                // every item's query tiles: one per wave
    const dim3 dgrid(a.meta.n_items, a.Hkv, a.nsplit_max * (unsigned)((queries_per_item_max + 63) / 64));
#define ATTN_MMA_R(D_, R_)                                                                        \
    do {                                                                                          \
        if (a.dma && bf) attn_dma_kernel<D_, DT_BF16, R_><<<dgrid, block, 0, st>>>(a);            \
        else if (a.dma) attn_dma_kernel<D_, DT_F16, R_><<<dgrid, block, 0, st>>>(a);              \
        else if (bf && one) attn_mma_kernel<D_, DT_BF16, 1, R_><<<grid, block, 0, st>>>(a);       \
        else if (bf) attn_mma_kernel<D_, DT_BF16, 2, R_><<<grid, block, 0, st>>>(a);              \
        else if (one) attn_mma_kernel<D_, DT_F16, 1, R_><<<grid, block, 0, st>>>(a);              \
        else attn_mma_kernel<D_, DT_F16, 2, R_><<<grid, block, 0, st>>>(a);                       \
    } while (0)
#define ATTN_MMA(D_)                                                                              \
    do {                                                                                          \
        if (a.dbg_logits) ATTN_MMA_R(D_, true);          /* test support: record queries and scores */ \
        else ATTN_MMA_R(D_, false);                                                               \
    } while (0)
    if (head_dim == 128) {
        if (!a.vector_path) ATTN_MMA(128);
        else if (wide) attn_kernel<128, 8><<<grid, block, 0, st>>>(a);
        else attn_kernel<128, 4><<<grid, block, 0, st>>>(a);
        attn_merge_kernel<128><<<mgrid, dim3(128), 0, st>>>(a);
    } else if (head_dim == 64) {
        if (!a.vector_path) ATTN_MMA(64);
        else if (wide) attn_kernel<64, 8><<<grid, block, 0, st>>>(a);
        else attn_kernel<64, 4><<<grid, block, 0, st>>>(a);
        attn_merge_kernel<64><<<mgrid, dim3(64), 0, st>>>(a);
    } else {
        return hipErrorInvalidValue;
    }
#undef ATTN_MMA
#undef ATTN_MMA_R
    return hipGetLastError();
}

// ------------------------------------------------------------------ prefill attention
//
// Causal attention of a prompt's rows (already in the cache) and the rows before
// them, for one layer of a one-slot state: cache rows are read where they lie,
// no beam table.  A workgroup takes 64 QTW consecutive query vectors (token i,
// head of the group) of one kv head and every key they see, so the result leaves
// it finished and normalized, as the o product's prepared input: no partials, no
// merge launch.  Eight waves: four query tiles (times QTW) by two key groups,
// which take alternate 32-key steps and are merged through LDS at the end.
// Scores, softmax and output as attn_dma_kernel (query as two cache-dtype terms,
// S^T = K Q^T, O^T += V^T P^T).  Each step's rows go through registers into one
// of two LDS buffers per group while the step before computes; a wave reads the
// step's K and V once for its QTW query tiles, and with one tile the LDS reads
// (1024 cycles for the eight waves' steps) take longer than the products (768),
// so QTW = 2 where the prompt has workgroups enough.  Bound by vector instructions
// (about 150 per tile and step beside 24 products) and the steps' barriers: 2048
// tokens of 32 x 128 heads 240 -> about 89 us a layer, 517 after 1536 170 -> 88.
// Masked rows and rows past the block's last query enter as zeros with a -inf
// score, and so, for each wave, do the rows of tokens past its last: a non-finite
// row reaches no token before its group of 16 (a wave's 16 QTW query vectors lie
// in one such group: QTW is 1 where an odd number of heads shares a kv head).
template <int D, int KVDT, int QTW>
__global__ __launch_bounds__(512, 2) void attn_pf_kernel(PfAttnArgs a) {
    constexpr int HALF = D / 2, NCH = D / 8, DB = D / 32, MB = D / 16, RB = 2 * D;
    constexpr int SB = AK * RB;                              // bytes of one step's K (or V)
    constexpr int NL = SB / 16 / 256;                        // 16-byte pieces per thread and step, K and V each
    static_assert(NL >= 1, "step geometry");
    __shared__ __attribute__((aligned(16))) uint8_t kv[2][2][2][SB];   // [key group][buffer][K, V]
    __shared__ float2 sml[4 * QTW][64];
    static_assert(sizeof(kv) >= (size_t)4 * QTW * MB * 1024, "merge staging");
    // (divisions and clamps leave uniform values in vector registers: readfirstlane
    // keeps what the buffer resources are made of scalar)
    const int g = __builtin_amdgcn_readfirstlane(blockIdx.x % a.Hkv);
    const int blk = __builtin_amdgcn_readfirstlane((int)(gridDim.x / a.Hkv - 1 - blockIdx.x / a.Hkv));   // longest first
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, qw = wave & 3, tg = tid & 255;
    const int ql = lane & 15, lg = lane >> 4;
    const int Hq = a.Hq, gs = Hq / a.Hkv;
    const int R = a.n * gs, r0 = blk * 64 * QTW;
    const int kend = __builtin_amdgcn_readfirstlane(a.P + (min(R, r0 + 64 * QTW) - 1) / gs + 1);   // keys the block's last query sees
    const int nsteps = (kend + AK - 1) / AK;
    const uint16_t* kh = a.kl + (size_t)g * a.cap * D;
    const uint16_t* vh = a.vl + (size_t)g * a.cap * D;

    // ---- step st of this key group: its pieces to registers, then (masked rows as
    // zeros) to LDS; piece u of thread tg is chunk (tg + 256 u) mod NCH of its key,
    // stored at that chunk ^ (key mod NCH)
    u32x4 rk[NL], rv[NL];
    uint32_t word = 0u;                                      // key mask of the step held in rk, rv
    auto ld = [&](int st) {
        const uint32_t bytes = __builtin_amdgcn_readfirstlane(max(0, min(AK, kend - AK * st)) * RB);   // later rows read as zeros
        const size_t base = (size_t)min(st, nsteps - 1) * AK * D;
        const __amdgpu_buffer_rsrc_t bk = buf_rsrc(kh + base, bytes), bv = buf_rsrc(vh + base, bytes);
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            // the piece's place is in the lane offset: the uniform offset takes no
            // part in the bounds check that zeroes the rows at and past kend
            rk[u] = buf_load16(bk, 16u * tg + 4096u * u, 0);
            rv[u] = buf_load16(bv, 16u * tg + 4096u * u, 0);
        }
        word = a.mask ? a.mask[min(st, nsteps - 1)] : ~0u;
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int idx = tg + 256 * u, key = idx / NCH, c = idx % NCH;
            u32x4 k = rk[u], v = rv[u];
            if (word != ~0u) {
                const bool in = (word >> key) & 1u;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    k[e] = in ? k[e] : 0u;
                    v[e] = in ? v[e] : 0u;
                }
            }
            const int at = key * RB + 16 * (c ^ (key % NCH));
            *(u32x4*)&kv[kg][buf][0][at] = k;
            *(u32x4*)&kv[kg][buf][1][at] = v;
        }
    };
    ld(kg);

    // ---- this wave's query tiles: rotated, scaled, split into rounded part and residual
    u32x4 qh[QTW][DB], qr[QTW][DB];
    int qtok[QTW];
    float base[QTW];                                         // what is subtracted from the scores (-inf: no key seen yet)
    float lsum[QTW];                                         // sums of this lane's probabilities (fp32, not rounded)
    f32x4_t nb[QTW];                                         // -base (0 before the first key), the score products' start
    f32x4_t o[QTW][MB];
#pragma unroll
    for (int u = 0; u < QTW; ++u) {
        const int r = r0 + 16 * (QTW * qw + u) + ql;
        const bool ok = r < R;
        const int i = ok ? r / gs : a.n - 1, h = g * gs + (ok ? r % gs : 0);   // the last row stands in past the end
        qtok[u] = i;
        base[u] = -INFINITY;
        lsum[u] = 0.f;
        nb[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        const float* qrow = a.qkv + (size_t)i * a.qkv_ld + (size_t)h * D;
        const float2* rp = a.rope + (size_t)a.pos[i] * HALF;
#pragma unroll
        for (int ib = 0; ib < DB; ++ib) {
            const int d0 = 32 * ib + 8 * lg;                 // dims d0 .. d0 + 7 lie in one rotary half
            const bool lo_half = d0 < HALF;
            float x[8], xp[8];
            float2 cs[8];
            __builtin_memcpy(x, qrow + d0, 32);
            __builtin_memcpy(xp, qrow + (lo_half ? d0 + HALF : d0 - HALF), 32);
            __builtin_memcpy(cs, rp + (lo_half ? d0 : d0 - HALF), 64);
            uint16_t hb[8], rb[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float y = (lo_half ? (x[e] * cs[e].x - xp[e] * cs[e].y) : (x[e] * cs[e].x + xp[e] * cs[e].y)) * a.qscale;
                hb[e] = kv_round<KVDT>(y);
                rb[e] = kv_round<KVDT>(y - kv_float<KVDT>(hb[e]));
            }
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) {
                qh[u][ib][w2] = (uint32_t)hb[2 * w2] | ((uint32_t)hb[2 * w2 + 1] << 16);
                qr[u][ib][w2] = (uint32_t)rb[2 * w2] | ((uint32_t)rb[2 * w2 + 1] << 16);
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) o[u][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    // the wave's first token: steps up to it are causal for all; and the keys up to
    // its last: later ones never meet this wave
    const int tok0 = __builtin_amdgcn_readfirstlane(min(R - 1, r0 + 16 * QTW * qw) / gs);
    const int kw = __builtin_amdgcn_readfirstlane(a.P + (min(R, r0 + 16 * QTW * (qw + 1)) - 1) / gs + 1);

    uint32_t cword = word;
    put(0);
    ld(kg + 2);
    for (int st = kg, it = 0; st - kg < nsteps; st += 2, ++it) {   // the same number of turns in both groups
        const int buf = it & 1;
        __syncthreads();                                     // this buffer is complete; the other one is free
        const uint32_t w0 = cword;                           // this step's key mask
        cword = word;
        put(buf ^ 1);
        ld(st + 4);
        const int seen = kw - AK * st;                       // keys of the step that some query of the wave may see (uniform)
        if (seen <= 0) continue;                             // (past the last step too)
        const uint8_t* kb = kv[kg][buf][0];
        const uint8_t* vb = kv[kg][buf][1];
        u32x4 kf0[DB], kf1[DB], vf[MB];
        f32x4_t s0[QTW], s1[QTW];
#pragma unroll
        for (int ib = 0; ib < DB; ++ib) {
            const int c = 4 * ib + lg;
            kf0[ib] = *(const u32x4*)&kb[ql * RB + 16 * (c ^ (ql % NCH))];
            kf1[ib] = *(const u32x4*)&kb[(16 + ql) * RB + 16 * (c ^ ((16 + ql) % NCH))];
        }
#pragma unroll
        for (int u = 0; u < QTW; ++u) {
            s0[u] = s1[u] = nb[u];
#pragma unroll
            for (int ib = 0; ib < DB; ++ib) {
                s0[u] = mma_kv<KVDT>(kf0[ib], qh[u][ib], s0[u]);
                s1[u] = mma_kv<KVDT>(kf1[ib], qh[u][ib], s1[u]);
                s0[u] = mma_kv<KVDT>(kf0[ib], qr[u][ib], s0[u]);
                s1[u] = mma_kv<KVDT>(kf1[ib], qr[u][ib], s1[u]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);                   // the value reads take the key fragments' registers
        // value fragments: read h gives keys 16 h + 4 lg + e; this lane supplies
        // key 16 h + 4 lg + ql / 4, dims 16 mb + 4 (ql mod 4) .. + 3
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            typedef short s16x4 __attribute__((ext_vector_type(4)));
            u32x2 p[2];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int key = 16 * hh + 4 * lg + (ql >> 2);
                const int d = 16 * mb + 4 * (ql & 3);
                const uint8_t* ad = vb + key * RB + 16 * ((d >> 3) ^ (key % NCH)) + 2 * (d & 7);
                p[hh] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                      (__attribute__((address_space(3))) s16x4*)ad));
            }
            vf[mb] = u32x4{p[0][0], p[0][1], p[1][0], p[1][1]};
        }
        if (seen < AK) {                                     // later tokens' values enter as zeros: 0 * inf would reach this wave
            u32x4 see;
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) {
                const int key = 16 * (w2 >> 1) + 4 * lg + 2 * (w2 & 1);
                see[w2] = key + 1 < seen ? ~0u : key < seen ? 0xFFFFu : 0u;
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) vf[mb] &= see;
        }
        const bool all = w0 == ~0u && AK * st + AK - 1 <= a.P + tok0;   // every key of the step is seen by every query (uniform)
        const int kbase = AK * st + 4 * lg;
#pragma unroll
        for (int u = 0; u < QTW; ++u) {
            float sv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) sv[e] = e < 4 ? s0[u][e] : s1[u][e - 4];
            if (!all) {
                const int last = a.P + qtok[u] - kbase;      // keys up to kbase + last are causal
                uint32_t vbits = w0 >> (4 * lg);
                asm volatile("" : "+v"(vbits));              // the bit tests stay inside the branch
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int ko = (e < 4) ? e : 12 + e;
                    sv[e] = (((vbits >> ko) & 1u) && ko <= last) ? sv[e] : -INFINITY;
                }
            }
            float mx = sv[0];
#pragma unroll
            for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sv[e]);
            // A step in which no query's largest score rises has no exchange between
            // lanes and no correction.  (Letting the base lag by up to 8 saved more,
            // but the largest key's probability was then rounded too: the error
            // against 64 bits grew by 3%.)
            if (__any(mx > (base[u] == -INFINITY ? -INFINITY : 0.f))) {
                float x0f, x1f;
                lane_pair_k(mx, 16, x0f, x1f);
                mx = fmaxf(x0f, x1f);
                lane_pair_k(mx, 32, x0f, x1f);
                mx = fmaxf(x0f, x1f);                        // the query's largest score of the step, less the old base
                // a first key sets the base; no key yet leaves it; else it only rises
                const bool first = base[u] == -INFINITY;
                const float up = first ? (mx == -INFINITY ? 0.f : mx) : fmaxf(mx, 0.f);
                const float corr = first ? 0.f : __builtin_amdgcn_exp2f(-up);
                base[u] = first ? mx : base[u] + up;
#pragma unroll
                for (int j = 0; j < 4; ++j) nb[u][j] -= up;
                lsum[u] *= corr;
#pragma unroll
                for (int e = 0; e < 8; ++e) sv[e] -= up;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) o[u][mb][jj] *= corr;
            }
            float pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) pv[e] = __builtin_amdgcn_exp2f(sv[e]);
            lsum[u] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
            u32x4 pb;
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) pb[w2] = kv_pack2<KVDT>(pv[2 * w2], pv[2 * w2 + 1]);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) o[u][mb] = mma_kv<KVDT>(vf[mb], pb, o[u][mb]);
        }
    }

    // ---- the two key groups' (base, sum, output) through LDS, then the o product's input
#pragma unroll
    for (int u = 0; u < QTW; ++u) {                          // a query's sum: the four lanes that hold its keys
        float x0f, x1f;
        lane_pair_k(lsum[u], 16, x0f, x1f);
        lsum[u] = x0f + x1f;
        lane_pair_k(lsum[u], 32, x0f, x1f);
        lsum[u] = x0f + x1f;
    }
    __syncthreads();                                         // no wave reads its step's rows any more
    f32x4_t* so = (f32x4_t*)&kv[0][0][0][0];                 // [4 QTW tiles][MB][64 lanes]
    if (kg == 1) {
#pragma unroll
        for (int u = 0; u < QTW; ++u) {
            sml[QTW * qw + u][lane] = float2{base[u], lsum[u]};
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) so[((QTW * qw + u) * MB + mb) * 64 + lane] = o[u][mb];
        }
    }
    __syncthreads();
    if (kg == 1) return;
#pragma unroll
    for (int u = 0; u < QTW; ++u) {
        const int r = r0 + 16 * (QTW * qw + u) + ql;
        const float2 ml = sml[QTW * qw + u][lane];
        const float mn = fmaxf(base[u], ml.x);               // finite: every query sees its own row
        const float f0 = __builtin_amdgcn_exp2f(base[u] - mn), f1 = __builtin_amdgcn_exp2f(ml.x - mn);
        const float inv = 1.0f / (lsum[u] * f0 + ml.y * f1);
        const int m = qtok[u], h = g * gs + r % gs;
        uint16_t* bp = a.bp + (size_t)(m >> 6) * 64 * a.kp;
        float* bc = a.bc + (size_t)(m >> 6) * 2 * a.kp;
#pragma unroll
        for (int mp = 0; mp < MB / 2; ++mp) {                // 32 dims: one correction
            float cs = 0.f;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int mb = 2 * mp + q, k = h * D + 16 * mb + 4 * lg;
                const f32x4_t ob = so[((QTW * qw + u) * MB + mb) * 64 + lane];
                uint16_t c[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float h16 = f16_to_f32(f32_to_f16((o[u][mb][j] * f0 + ob[j] * f1) * inv));
                    cs += bp_corr(h16, j);
                    c[j] = bp_code(h16, j);
                }
                if (r < R) __builtin_memcpy(__builtin_assume_aligned(bp + bp_index(m & 63, k), 8), c, 8);
            }
            float x0f, x1f;
            lane_pair_k(cs, 16, x0f, x1f);
            cs = x0f + x1f;
            lane_pair_k(cs, 32, x0f, x1f);
            cs = x0f + x1f;
            if (r < R && lg == 0) bc[bc_index(m & 63, h * D + 32 * mp)] = cs;
        }
    }
}

hipError_t launch_attention_pf(const PfAttnArgs& a, int head_dim, int n_cus, hipStream_t st) {
    if (a.n < 1 || a.Hkv < 1 || a.Hq % a.Hkv || a.kp < a.Hq * head_dim || a.kp % 128) return hipErrorInvalidValue;
    const size_t R = (size_t)a.n * (a.Hq / a.Hkv);
    // one workgroup runs per CU; two query tiles per wave take about 5/3 of one
    // tile's time a step, so they pay where they save a round of workgroups
    const size_t w1 = (R + 63) / 64 * a.Hkv, w2 = (R + 127) / 128 * a.Hkv;
    const bool two = a.Hq / a.Hkv % 2 == 0 && 5 * ((w2 + n_cus - 1) / n_cus) <= 3 * ((w1 + n_cus - 1) / n_cus);
    const dim3 grid((unsigned)((R + (two ? 127 : 63)) / (two ? 128 : 64) * a.Hkv)), block(512);
    const bool bf = a.kv_dt == DT_BF16;
#define ATTN_PF(D_)                                                                               \
    do {                                                                                          \
        if (bf && two) attn_pf_kernel<D_, DT_BF16, 2><<<grid, block, 0, st>>>(a);                 \
        else if (bf) attn_pf_kernel<D_, DT_BF16, 1><<<grid, block, 0, st>>>(a);                   \
        else if (two) attn_pf_kernel<D_, DT_F16, 2><<<grid, block, 0, st>>>(a);                   \
        else attn_pf_kernel<D_, DT_F16, 1><<<grid, block, 0, st>>>(a);                            \
    } while (0)
    if (head_dim == 128) ATTN_PF(128);
    else if (head_dim == 64) ATTN_PF(64);
    else return hipErrorInvalidValue;
#undef ATTN_PF
    return hipGetLastError();
}

// ------------------------------------------------------------------ fill

// p[0 .. n) = v.
__global__ __launch_bounds__(256) void fill_u32_kernel(uint32_t* __restrict__ p, size_t n, uint32_t v) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
    fill_u32_kernel<<<blocks, 256, 0, st>>>(p, n, v);
    return hipGetLastError();
}

// ------------------------------------------------------------------ KV state kernels

__global__ void table_gather_kernel(const int16_t* __restrict__ src, int16_t* __restrict__ dst, const int* __restrict__ beam,
                                    int S, int cap, int P) {
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= (size_t)S * P) return;
    const int b = (int)(idx / P), j = (int)(idx % P);
    dst[(size_t)b * cap + j] = src[(size_t)beam[b] * cap + j];
}

hipError_t launch_table_gather(const int16_t* src, int16_t* dst, const int* beam, int S, int cap, int P, hipStream_t st) {
    const size_t n = (size_t)S * P;
    if (n == 0) return hipSuccess;
    table_gather_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(src, dst, beam, S, cap, P);
    return hipGetLastError();
}

// Rows [L][S][Hkv][n][D] of k, v to physical rows P..P+n-1 of every slot; the
// slots' table entries there become their own index.  One thread moves 16
// bytes of K and of V (D is a multiple of 8).
__global__ __launch_bounds__(256) void kv_append_kernel(uint16_t* __restrict__ kc, uint16_t* __restrict__ vc,
                                                        int16_t* __restrict__ table, const uint16_t* __restrict__ k,
                                                        const uint16_t* __restrict__ v, int L, int S, int Hkv, int cap, int D,
                                                        int P, int n) {
    const int tpr = D / 8;
    const size_t total = (size_t)L * S * Hkv * n * tpr;
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= total) return;
    size_t rem = idx;
    const int e = (int)(rem % tpr); rem /= tpr;
    const int i = (int)(rem % n); rem /= n;
    const int g = (int)(rem % Hkv); rem /= Hkv;
    const int b = (int)(rem % S); rem /= S;
    const int l = (int)rem;
    const size_t dst = ((((size_t)l * S + b) * Hkv + g) * cap + (P + i)) * D + 8 * e;
    *(uint4*)(kc + dst) = *(const uint4*)(k + 8 * idx);
    *(uint4*)(vc + dst) = *(const uint4*)(v + 8 * idx);
    if (l == 0 && g == 0 && e == 0) table[(size_t)b * cap + P + i] = (int16_t)b;
}

hipError_t launch_kv_append(uint16_t* kc, uint16_t* vc, int16_t* table, const uint16_t* k, const uint16_t* v,
                            int L, int S, int Hkv, int cap, int D, int P, int n, hipStream_t st) {
    if (D % 8) return hipErrorInvalidValue;
    const size_t total = (size_t)L * S * Hkv * n * (D / 8);
    if (total == 0) return hipSuccess;
    kv_append_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st>>>(kc, vc, table, k, v, L, S, Hkv, cap, D, P, n);
    return hipGetLastError();
}

__global__ void kv_read_kernel(const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, const int16_t* __restrict__ table,
                               int layer, int slot, int start, int count, int S, int Hkv, int cap, int D,
                               uint16_t* __restrict__ k_out, uint16_t* __restrict__ v_out) {
    const size_t total = (size_t)Hkv * count * D;
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int d = (int)(idx % D);
    const int c = (int)((idx / D) % count);
    const int g = (int)(idx / ((size_t)D * count));
    const int j = start + c;
    const int ps = table[(size_t)slot * cap + j];
    const size_t src = ((((size_t)layer * S + ps) * Hkv + g) * cap + j) * D + d;
    k_out[idx] = kc[src];
    v_out[idx] = vc[src];
}

hipError_t launch_kv_read(const uint16_t* kc, const uint16_t* vc, const int16_t* table, int layer, int slot,
                          int start, int count, int S, int Hkv, int cap, int D, uint16_t* k_out, uint16_t* v_out,
                          hipStream_t st) {
    const size_t total = (size_t)Hkv * count * D;
    if (total == 0) return hipSuccess;
    kv_read_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st>>>(kc, vc, table, layer, slot, start, count,
                                                                                  S, Hkv, cap, D, k_out, v_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ compaction and capture

// dst row i of slot b (for every layer and kv head) = the row src[b][i] of the
// slot's view, read through the beam table (physical slot table[b][j] holds
// row j); src[b][i] < 0 writes a zero row.  One thread moves 16 bytes of K and
// 16 of V; a row is D / 8 consecutive threads, so a wave's loads and stores
// cover whole rows.  dst rows of one (layer, slot, kv head) are dst_stride
// rows apart.
__global__ __launch_bounds__(256) void kv_gather_rows_kernel(const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
                                                             const int16_t* __restrict__ table, const int* __restrict__ src,
                                                             int L, int S, int Hkv, int cap, int D, int Pn, int dst_stride,
                                                             uint16_t* __restrict__ k_dst, uint16_t* __restrict__ v_dst) {
    const int tpr = D / 8;
    const size_t rows = (size_t)L * S * Hkv * Pn;
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= rows * tpr) return;
    const int e = (int)(idx % tpr);
    size_t r = idx / tpr;
    const int i = (int)(r % Pn); r /= Pn;
    const int g = (int)(r % Hkv); r /= Hkv;
    const int b = (int)(r % S);
    const int l = (int)(r / S);
    const size_t dst = ((((size_t)l * S + b) * Hkv + g) * dst_stride + i) * D + 8 * e;
    const int j = src[(size_t)b * Pn + i];
    uint4 kv = {0u, 0u, 0u, 0u}, vv = {0u, 0u, 0u, 0u};
    if (j >= 0) {
        const int ps = table[(size_t)b * cap + j];
        const size_t so = ((((size_t)l * S + ps) * Hkv + g) * cap + j) * D + 8 * e;
        kv = *(const uint4*)(kc + so);
        vv = *(const uint4*)(vc + so);
    }
    *(uint4*)(k_dst + dst) = kv;
    *(uint4*)(v_dst + dst) = vv;
}

hipError_t launch_kv_gather_rows(const uint16_t* kc, const uint16_t* vc, const int16_t* table, const int* src, int L, int S,
                                 int Hkv, int cap, int D, int Pn, int dst_stride, uint16_t* k_dst, uint16_t* v_dst,
                                 hipStream_t st) {
    if (D % 8) return hipErrorInvalidValue;
    const size_t n = (size_t)L * S * Hkv * Pn * (D / 8);
    if (n == 0) return hipSuccess;
    kv_gather_rows_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(kc, vc, table, src, L, S, Hkv, cap, D,
                                                                                    Pn, dst_stride, k_dst, v_dst);
    return hipGetLastError();
}

// In-place compaction of one cache (K or V): row i of slot b becomes the row
// src[b][i] of the slot's view (through the beam table), or zero where
// src[b][i] < 0.  src[b][i] >= i (kept rows in ascending order), so a row read
// for destination i is never a destination below i.  One workgroup owns one
// column slice (KC_SLICES per row) of one (layer, kv head, K or V) for every
// slot and walks the destination rows in chunks of `chunk` positions:
//  - all of a chunk's loads complete before any of its stores (the wait and
//    the barrier before the stores);
//  - the loads of chunk c + 1 are issued before the stores of chunk c: they
//    read rows at or above the first position of chunk c + 1, the stores of
//    chunk c write rows below it, so the two never touch the same element;
//  - rows read by later chunks lie at or above their destinations, above
//    every row written so far.
// So no element is overwritten before every read of it.  Column slices are
// independent (a row's slice moves with the row).
constexpr int KC_THREADS = 512;
constexpr int KC_PIECES = 4;
constexpr int KC_SLICES = 2;

struct KcChunk {
    uint4 v[KC_PIECES];
};

__device__ __forceinline__ void kc_load(const uint16_t* c, const int16_t* __restrict__ table, const int* __restrict__ src,
                                        int l, int g, int S, int Hkv, int cap, int D, int Pn, int pps, int col0, int i0,
                                        int cn, KcChunk& ch) {
    const int pieces = S * cn * pps;
#pragma unroll
    for (int k = 0; k < KC_PIECES; ++k) {
        const int p = threadIdx.x + k * KC_THREADS;
        ch.v[k] = make_uint4(0u, 0u, 0u, 0u);
        if (p < pieces) {
            const int r = p / pps;
            const int b = r / cn;
            const int i = i0 + r % cn;
            const int j = src[(size_t)b * Pn + i];
            if (j >= 0) {
                const int ps = table[(size_t)b * cap + j];
                ch.v[k] = *(const uint4*)(c + ((((size_t)l * S + ps) * Hkv + g) * cap + j) * D + col0 + 8 * (p % pps));
            }
        }
    }
}

__device__ __forceinline__ void kc_store(uint16_t* c, int l, int g, int S, int Hkv, int cap, int D, int pps, int col0,
                                         int i0, int cn, const KcChunk& ch) {
    const int pieces = S * cn * pps;
#pragma unroll
    for (int k = 0; k < KC_PIECES; ++k) {
        const int p = threadIdx.x + k * KC_THREADS;
        if (p < pieces) {
            const int r = p / pps;
            const int b = r / cn;
            const int i = i0 + r % cn;
            *(uint4*)(c + ((((size_t)l * S + b) * Hkv + g) * cap + i) * D + col0 + 8 * (p % pps)) = ch.v[k];
        }
    }
}

__global__ __launch_bounds__(KC_THREADS) void kv_compact_kernel(uint16_t* kc, uint16_t* vc, const int16_t* __restrict__ table,
                                                                const int* __restrict__ src, int S, int Hkv, int cap,
                                                                int D, int Pn, int chunk) {
    const int slice = blockIdx.x % KC_SLICES;
    const int u = blockIdx.x / KC_SLICES;
    const int l = u / (2 * Hkv);
    const int g = (u / 2) % Hkv;
    uint16_t* c = (u & 1) ? vc : kc;
    const int pps = D / 8 / KC_SLICES;                       // 16-byte pieces of a row slice
    const int col0 = slice * pps * 8;                        // first element of the slice
    KcChunk a, b;
    kc_load(c, table, src, l, g, S, Hkv, cap, D, Pn, pps, col0, 0, min(chunk, Pn), a);
    for (int i0 = 0; i0 < Pn; i0 += 2 * chunk) {
        // chunk at i0 (in a), then chunk at i0 + chunk (in b)
        const int i1 = i0 + chunk, i2 = i0 + 2 * chunk;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's accesses have completed
        __syncthreads();                                     // and so have every other wave's
        if (i1 < Pn) kc_load(c, table, src, l, g, S, Hkv, cap, D, Pn, pps, col0, i1, min(chunk, Pn - i1), b);
        kc_store(c, l, g, S, Hkv, cap, D, pps, col0, i0, min(chunk, Pn - i0), a);
        if (i1 >= Pn) break;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (i2 < Pn) kc_load(c, table, src, l, g, S, Hkv, cap, D, Pn, pps, col0, i2, min(chunk, Pn - i2), a);
        kc_store(c, l, g, S, Hkv, cap, D, pps, col0, i1, min(chunk, Pn - i1), b);
    }
}

hipError_t launch_kv_compact(uint16_t* kc, uint16_t* vc, const int16_t* table, const int* src, int L, int S, int Hkv,
                             int cap, int D, int Pn, hipStream_t st) {
    if (D % (8 * KC_SLICES)) return hipErrorInvalidValue;
    if (Pn == 0 || L == 0) return hipSuccess;
    const int pps = D / 8 / KC_SLICES;
    if ((long)S * pps > (long)KC_THREADS * KC_PIECES) return hipErrorInvalidValue;   // a chunk holds every slot's row
    const int chunk = KC_THREADS * KC_PIECES / (S * pps);
    kv_compact_kernel<<<dim3((unsigned)(L * Hkv * 2 * KC_SLICES)), dim3(KC_THREADS), 0, st>>>(kc, vc, table, src, S, Hkv,
                                                                                             cap, D, Pn, chunk);
    return hipGetLastError();
}

// ------------------------------------------------------------------ top-1 of the LM head

// One workgroup per row: the tiles' (max, index, sum of exp(v - max)) reduced
// in a fixed order (strided per thread, then a tree), so the result does not
// depend on timing.  Ties on the value take the smallest index.
__global__ __launch_bounds__(256) void top1_merge_kernel(const float4* __restrict__ part, int ntiles, int32_t* __restrict__ token,
                                                         float* __restrict__ p, float* __restrict__ logit) {
    __shared__ float smx[256];
    __shared__ int sarg[256];
    __shared__ float sse[256];
    const int m = blockIdx.x, tid = threadIdx.x;
    const float4* row = part + (size_t)m * ntiles;
    float mx = -INFINITY;
    int arg = INT_MAX;
    for (int t = tid; t < ntiles; t += 256) {
        const float4 e = row[t];
        const int ei = __float_as_int(e.y);
        if (e.x > mx || (e.x == mx && ei < arg)) {
            mx = e.x;
            arg = ei;
        }
    }
    smx[tid] = mx;
    sarg[tid] = arg;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) {
            const float x2 = smx[tid + o];
            const int a2 = sarg[tid + o];
            if (x2 > smx[tid] || (x2 == smx[tid] && a2 < sarg[tid])) {
                smx[tid] = x2;
                sarg[tid] = a2;
            }
        }
        __syncthreads();
    }
    const float gmx = smx[0];
    float se = 0.f;
    for (int t = tid; t < ntiles; t += 256) {
        const float4 e = row[t];
        se += e.z * expf(e.x - gmx);
    }
    sse[tid] = se;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) sse[tid] += sse[tid + o];
        __syncthreads();
    }
    if (tid == 0) {
        token[m] = sarg[0];
        p[m] = 1.0f / sse[0];
        if (logit) logit[m] = gmx;
    }
}

hipError_t launch_top1_merge(const float4* part, int M, int ntiles, int32_t* token, float* p, float* logit, hipStream_t st) {
    if (M < 1 || ntiles < 1) return hipErrorInvalidValue;
    top1_merge_kernel<<<dim3((unsigned)M), dim3(256), 0, st>>>(part, ntiles, token, p, logit);
    return hipGetLastError();
}

// ------------------------------------------------------------------ stage-0 embedding gather

// Row m of out = row ids[m] of the token table [vocab][row_elems], copied
// unchanged; an id outside [0, vocab) gives a zero row and sets *err.  One
// workgroup per row; T is the copy width (16 bytes when both pointers allow).
template <class T>
__global__ __launch_bounds__(256) void embed_gather_kernel(const T* __restrict__ table, const int32_t* __restrict__ ids,
                                                           int vocab, int row_elems, T* __restrict__ out,
                                                           unsigned* __restrict__ err) {
    const int m = blockIdx.x;
    const int id = ids[m];
    T* dst = out + (size_t)m * row_elems;
    if (id < 0 || id >= vocab) {
        for (int i = threadIdx.x; i < row_elems; i += 256) dst[i] = T(0);
        if (threadIdx.x == 0) atomicOr(err, 1u);
        return;
    }
    const T* src = table + (size_t)id * row_elems;
    for (int i = threadIdx.x; i < row_elems; i += 256) dst[i] = src[i];
}

hipError_t launch_embed_gather(const uint16_t* table, const int32_t* ids, int n, int vocab, int H, uint16_t* out,
                               unsigned* err, hipStream_t st) {
    if (n < 1 || vocab < 1 || H < 1) return hipErrorInvalidValue;
    if (H % 8 == 0 && ((uintptr_t)table & 15) == 0 && ((uintptr_t)out & 15) == 0)
        embed_gather_kernel<u32x4><<<dim3((unsigned)n), dim3(256), 0, st>>>((const u32x4*)table, ids, vocab, H / 8,
                                                                          (u32x4*)out, err);
    else
        embed_gather_kernel<uint16_t><<<dim3((unsigned)n), dim3(256), 0, st>>>(table, ids, vocab, H, out, err);
    return hipGetLastError();
}

// The k and v rows of n prompt rows (q|k|v results [n][ld], fp32) of a one-slot
// state to cache rows P .. P + n - 1 of one layer: k rotated at the row's
// position (rotate-half pairing), both rounded to the cache dtype.  One thread
// per (row, kv head, dimension).
__global__ __launch_bounds__(256) void kv_rope_append_kernel(const float* __restrict__ qkv, int ld, const int* __restrict__ pos,
                                                             const float2* __restrict__ rope, int n, int P, int Hq, int Hkv,
                                                             int D, uint16_t* __restrict__ kl, uint16_t* __restrict__ vl,
                                                             int cap, int16_t* __restrict__ table, int kv_dt) {
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= (size_t)n * Hkv * D) return;
    const int d = (int)(idx % D);
    const int g = (int)((idx / D) % Hkv);
    const int i = (int)(idx / ((size_t)D * Hkv));
    const int half = D / 2;
    const float* krow = qkv + (size_t)i * ld + (size_t)(Hq + g) * D;
    const float* vrow = qkv + (size_t)i * ld + (size_t)(Hq + Hkv + g) * D;
    const bool lo_half = d < half;
    const float xk = krow[d];
    const float xp = lo_half ? krow[d + half] : krow[d - half];
    const float2 cs = rope[(size_t)pos[i] * half + (lo_half ? d : d - half)];
    const float y = lo_half ? (xk * cs.x - xp * cs.y) : (xk * cs.x + xp * cs.y);
    const size_t off = ((size_t)g * cap + P + i) * D + d;
    kl[off] = to_half_bits(y, kv_dt);
    vl[off] = to_half_bits(vrow[d], kv_dt);
    if (table && g == 0 && d == 0) table[P + i] = 0;
}

hipError_t launch_kv_rope_append(const float* qkv, int ld, const int* pos, const float2* rope, int n, int P, int Hq, int Hkv,
                                 int D, uint16_t* kl, uint16_t* vl, int cap, int16_t* table, int kv_dt, hipStream_t st) {
    const size_t t = (size_t)n * Hkv * D;
    if (t == 0) return hipSuccess;
    kv_rope_append_kernel<<<dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st>>>(qkv, ld, pos, rope, n, P, Hq, Hkv, D, kl, vl,
                                                                                    cap, table, kv_dt);
    return hipGetLastError();
}

// table[b][j] = b for j < n: every slot reads its own rows.
__global__ void table_identity_kernel(int16_t* __restrict__ table, int S, int cap, int n) {
    const size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (idx >= (size_t)S * n) return;
    const int b = (int)(idx / n), j = (int)(idx % n);
    table[(size_t)b * cap + j] = (int16_t)b;
}

hipError_t launch_table_identity(int16_t* table, int S, int cap, int n, hipStream_t st) {
    const size_t t = (size_t)S * n;
    if (t == 0) return hipSuccess;
    table_identity_kernel<<<dim3((unsigned)((t + 255) / 256)), dim3(256), 0, st>>>(table, S, cap, n);
    return hipGetLastError();
}

}  // namespace stg
