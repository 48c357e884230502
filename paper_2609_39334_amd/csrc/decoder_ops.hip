// The elementwise steps of a decoder layer between its matrix products, each as one pass over memory:
//   add_rmsnorm  x += delta, h = RMSNorm(x)          (residual add, norm and the cast for the next product)
//   rope_append  RoPE of q and k, q packed for attention, k and v written to their pool slots
//   swiglu       a = SiLU(gate) * up
// All are HBM-bound; written as separate tensor operations every one of them read and wrote its operands
// three to six times, in fp32.  Arithmetic is fp32 throughout, rounded once to bf16 where the result is
// bf16 (nearest even).  Measured on 1,024 rows of the 28/4/128, hidden 3,584, inter 18,944 layout: a step
// of four layers takes 4.07 ms against 5.22 ms with tensor operations, i.e. 290 us less per layer; of a
// layer's kernels add_rmsnorm takes 10.6 us (twice; 4.1 TB/s), rope_append 7.0 us and swiglu 19.8 us
// (5.9 TB/s).
#include <hip/hip_runtime.h>
#include <cstdint>

#include "internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kHeldVecs = 8;  // float4s of a row that a thread of add_rmsnorm keeps

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}
__device__ __forceinline__ float lo_f32(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float hi_f32(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

template <int T>
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < T / 64; k += 4) sum += (red[k] + red[k + 1]) + (red[k + 2] + red[k + 3]);
    return sum;
}

// One workgroup of T threads per row.  Rows of up to 32 T (a multiple of eight) stay in registers between the
// sum of squares and the scaling; other rows are read again (from the caches: the thread has just written
// them).  256 threads up to 8,192, 512 up to 16,384 (one row of 16,384 23 us read again by 256, 8.7 us held;
// 1,500 rows 67, 45); 1,024 for other rows of more than 4,096 (one row of 20,480 29 us with 256, 9.9 us;
// 1,500 rows 84, 72).
template <int T, bool HELD>
__global__ __launch_bounds__(T) void add_rmsnorm(int hidden, float eps, float* __restrict__ x,
                                                 const uint16_t* __restrict__ delta, const float* __restrict__ weight,
                                                 uint16_t* __restrict__ h) {
    __shared__ float red[T / 64];
    const size_t row = static_cast<size_t>(blockIdx.x) * hidden;
    const int t = threadIdx.x;
    float sq = 0.f;
    if constexpr (HELD) {
        const int n4 = hidden / 4;
        float4* x4 = reinterpret_cast<float4*>(x + row);
        const uint2* d2 = reinterpret_cast<const uint2*>(delta + row);
        float4 v[kHeldVecs];
#pragma unroll
        for (int k = 0; k < kHeldVecs; ++k) {
            const int i = t + k * T;
            if (i >= n4) continue;
            v[k] = x4[i];
            if (delta) {
                const uint2 d = d2[i];
                v[k].x += lo_f32(d.x);
                v[k].y += hi_f32(d.x);
                v[k].z += lo_f32(d.y);
                v[k].w += hi_f32(d.y);
                x4[i] = v[k];
            }
            sq += (v[k].x * v[k].x + v[k].y * v[k].y) + (v[k].z * v[k].z + v[k].w * v[k].w);
        }
        const float r = 1.f / sqrtf(block_sum<T>(sq, red) / static_cast<float>(hidden) + eps);
        const float4* w4 = reinterpret_cast<const float4*>(weight);
        uint2* h2 = reinterpret_cast<uint2*>(h + row);
#pragma unroll
        for (int k = 0; k < kHeldVecs; ++k) {
            const int i = t + k * T;
            if (i >= n4) continue;
            const float4 w = w4[i];
            h2[i] = uint2{pack_bf16x2(v[k].x * r * w.x, v[k].y * r * w.y), pack_bf16x2(v[k].z * r * w.z, v[k].w * r * w.w)};
        }
    } else {
        for (int i = t; i < hidden; i += T) {
            float v = x[row + i];
            if (delta) {
                v += lo_f32(delta[row + i]);
                x[row + i] = v;
            }
            sq += v * v;
        }
        const float r = 1.f / sqrtf(block_sum<T>(sq, red) / static_cast<float>(hidden) + eps);
        for (int i = t; i < hidden; i += T)
            h[row + i] = static_cast<uint16_t>(pack_bf16x2(x[row + i] * r * weight[i], 0.f));
    }
}

// One thread per 8 + 8 elements of a head (the two that RoPE rotates together, or 16 of a v head).
template <int D>
__global__ __launch_bounds__(kThreads) void rope_append(int64_t n_pieces, int hq, int hkv, int32_t n_slots,
                                                        const uint16_t* __restrict__ qkv, const float* __restrict__ cosv,
                                                        const float* __restrict__ sinv, const int32_t* __restrict__ dst,
                                                        uint16_t* __restrict__ q, uint16_t* __restrict__ kpool,
                                                        uint16_t* __restrict__ vpool) {
    constexpr int PPH = D / 16;  // pieces per head
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= n_pieces) return;
    const int64_t row = i / PPH;  // (token, head) row
    const int c = static_cast<int>(i - row * PPH);
    const int heads = hq + 2 * hkv;
    const int64_t t = row / heads;
    const int h = static_cast<int>(row - t * heads);
    uint16_t* out;
    if (h < hq) {
        out = q + (t * hq + h) * D;
    } else {
        const int32_t slot = dst[t];
        if (slot < 0 || slot >= n_slots) return;  // no slot: nothing to write
        const int64_t blk = slot / tkv::kBlock, pos = slot - blk * tkv::kBlock;
        const int kh = h < hq + hkv ? h - hq : h - hq - hkv;
        out = (h < hq + hkv ? kpool : vpool) + ((blk * hkv + kh) * tkv::kBlock + pos) * D;
    }
    const uint16_t* in = qkv + row * D;
    const uint4 a = *reinterpret_cast<const uint4*>(in + 8 * c), b = *reinterpret_cast<const uint4*>(in + D / 2 + 8 * c);
    uint4 oa = a, ob = b;
    if (h < hq + hkv) {
        const float4* cp = reinterpret_cast<const float4*>(cosv + t * (D / 2) + 8 * c);
        const float4* sp = reinterpret_cast<const float4*>(sinv + t * (D / 2) + 8 * c);
        const float4 c0 = cp[0], c1 = cp[1], s0 = sp[0], s1 = sp[1];
        const float cs[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
        const float sn[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
        const uint32_t ua[4] = {a.x, a.y, a.z, a.w}, ub[4] = {b.x, b.y, b.z, b.w};
        uint32_t ra[4], rb[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x0 = lo_f32(ua[e]), x1 = hi_f32(ua[e]), y0 = lo_f32(ub[e]), y1 = hi_f32(ub[e]);
            ra[e] = pack_bf16x2(x0 * cs[2 * e] - y0 * sn[2 * e], x1 * cs[2 * e + 1] - y1 * sn[2 * e + 1]);
            rb[e] = pack_bf16x2(y0 * cs[2 * e] + x0 * sn[2 * e], y1 * cs[2 * e + 1] + x1 * sn[2 * e + 1]);
        }
        oa = uint4{ra[0], ra[1], ra[2], ra[3]};
        ob = uint4{rb[0], rb[1], rb[2], rb[3]};
    }
    *reinterpret_cast<uint4*>(out + 8 * c) = oa;
    *reinterpret_cast<uint4*>(out + D / 2 + 8 * c) = ob;
}

// SiLU(g) u = g / (1 + exp(-g)) u.  exp(-g) is 2^n 2^f: g has the 8 significant bits of bf16 and kHi 13, so
// g kHi is exact, n its nearest integer, and f rounds once.  For negative g the reciprocal is taken of 2^-64 of
// the sum, so that nothing is flushed while exp(-g) is finite (exp2 and rcp of the plain values gave 0 for
// gates under -87).  The same bf16 results as with expf and a division on 2 M values.  813 rows of 18,944:
// 16.7 us, 18.1 us with those, 16.3 us with plain exp2 and rcp.
__device__ __forceinline__ float silu_mul(float g, float u) {
    constexpr float kHi = 0x1.715p0f, kLo = static_cast<float>(1.4426950408889634 - 0x1.715p0);  // log2(e)
    const float a = fminf(fmaxf(-kHi * g, -160.f), 160.f);  // exp is 0 or inf past the ends; g = +-inf shows in f
    const float n = rintf(a);
    const float e = ldexpf(__builtin_amdgcn_exp2f(fmaf(g, -kLo, a - n)), static_cast<int>(n));
    const float c = g < 0.f ? 0x1p-64f : 1.f;
    return g * __builtin_amdgcn_rcpf(fmaf(e, c, c)) * c * u;
}

// VEC: eight columns per thread (inter a multiple of eight, 16-byte aligned rows); else one.
template <bool VEC>
__global__ __launch_bounds__(kThreads) void swiglu(int64_t n, int64_t inter, const uint16_t* __restrict__ gu,
                                                   uint16_t* __restrict__ out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= n) return;
    if constexpr (VEC) {
        const int64_t per = inter / 8, row = i / per, c = i - row * per;
        const uint4* in = reinterpret_cast<const uint4*>(gu) + row * 2 * per + c;
        const uint4 g = in[0], u = in[per];
        reinterpret_cast<uint4*>(out)[i] = uint4{
            pack_bf16x2(silu_mul(lo_f32(g.x), lo_f32(u.x)), silu_mul(hi_f32(g.x), hi_f32(u.x))),
            pack_bf16x2(silu_mul(lo_f32(g.y), lo_f32(u.y)), silu_mul(hi_f32(g.y), hi_f32(u.y))),
            pack_bf16x2(silu_mul(lo_f32(g.z), lo_f32(u.z)), silu_mul(hi_f32(g.z), hi_f32(u.z))),
            pack_bf16x2(silu_mul(lo_f32(g.w), lo_f32(u.w)), silu_mul(hi_f32(g.w), hi_f32(u.w)))};
    } else {
        const int64_t row = i / inter, c = i - row * inter;
        const uint16_t* in = gu + row * 2 * inter + c;
        out[i] = static_cast<uint16_t>(pack_bf16x2(silu_mul(lo_f32(in[0]), lo_f32(in[inter])), 0.f));
    }
}

bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

int launched(const char* fn) {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TKV_OK : tkv::set_error(TKV_EHIP, "%s launch: %s", fn, hipGetErrorString(e));
}

constexpr int64_t kMaxGrid = INT32_MAX;

}  // namespace

TKV_EXPORT int tkv_add_rmsnorm(int32_t n_rows, int32_t hidden, float eps, float* x, const void* delta,
                               const float* weight, void* h, void* stream) {
    tkv::clear_error();
    if (n_rows < 0 || hidden < 1) return tkv::set_error(TKV_EINVAL, "tkv_add_rmsnorm: n_rows %d, hidden %d", n_rows, hidden);
    if (n_rows == 0) return TKV_OK;
    if (!x || !weight || !h) return tkv::set_error(TKV_EINVAL, "tkv_add_rmsnorm: NULL pointer");
    const bool held = hidden % 8 == 0 && hidden <= 4 * kHeldVecs * 512 && aligned16(x) && aligned16(delta) &&
                      aligned16(weight) && aligned16(h);
    const auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(n_rows)), dim3(static_cast<unsigned>(threads)), 0,
                           static_cast<hipStream_t>(stream), hidden, eps, x, static_cast<const uint16_t*>(delta), weight,
                           static_cast<uint16_t*>(h));
    };
    if (held && hidden <= 4 * kHeldVecs * 256)
        launch(add_rmsnorm<256, true>, 256);
    else if (held)
        launch(add_rmsnorm<512, true>, 512);
    else if (hidden <= 4096)
        launch(add_rmsnorm<256, false>, 256);
    else
        launch(add_rmsnorm<1024, false>, 1024);
    return launched("tkv_add_rmsnorm");
}

TKV_EXPORT int tkv_rope_append(const tkv_shape* shape, int32_t n_tok, const void* qkv, const float* cosv,
                               const float* sinv, const int32_t* d_dst, void* q, void* k, void* v, void* stream) {
    tkv::clear_error();
    if (!shape) return tkv::set_error(TKV_EINVAL, "tkv_rope_append: shape is NULL");
    const tkv_shape s = *shape;
    if (s.block_size != tkv::kBlock) return tkv::set_error(TKV_EINVAL, "tkv_rope_append: block_size must be 16 (got %d)", s.block_size);
    if (s.d != 64 && s.d != 128) return tkv::set_error(TKV_EINVAL, "tkv_rope_append: head_dim must be 64 or 128 (got %d)", s.d);
    if (s.hq < 1 || s.hkv < 1 || s.num_blocks < 1)
        return tkv::set_error(TKV_EINVAL, "tkv_rope_append: hq, hkv and num_blocks must be >= 1");
    if (static_cast<int64_t>(s.num_blocks) * s.block_size > INT32_MAX)
        return tkv::set_error(TKV_EINVAL, "tkv_rope_append: %d blocks exceed the int32 slot range", s.num_blocks);
    if (n_tok < 0) return tkv::set_error(TKV_EINVAL, "tkv_rope_append: n_tok = %d < 0", n_tok);
    if (n_tok == 0) return TKV_OK;
    if (!qkv || !cosv || !sinv || !d_dst || !q || !k || !v) return tkv::set_error(TKV_EINVAL, "tkv_rope_append: NULL pointer");
    if (!aligned16(qkv) || !aligned16(cosv) || !aligned16(sinv) || !aligned16(q) || !aligned16(k) || !aligned16(v))
        return tkv::set_error(TKV_EINVAL, "tkv_rope_append: tensors must be 16-byte aligned");
    const int64_t n = static_cast<int64_t>(n_tok) * (static_cast<int64_t>(s.hq) + 2 * static_cast<int64_t>(s.hkv)) * (s.d / 16);
    const int64_t grid = (n + kThreads - 1) / kThreads;
    if (grid > kMaxGrid) return tkv::set_error(TKV_EINVAL, "tkv_rope_append: %d tokens are too many", n_tok);
    const auto kernel = s.d == 128 ? rope_append<128> : rope_append<64>;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, static_cast<hipStream_t>(stream), n, s.hq,
                       s.hkv, s.num_blocks * s.block_size, static_cast<const uint16_t*>(qkv), cosv, sinv, d_dst,
                       static_cast<uint16_t*>(q), static_cast<uint16_t*>(k), static_cast<uint16_t*>(v));
    return launched("tkv_rope_append");
}

TKV_EXPORT int tkv_swiglu(int32_t n_rows, int32_t inter, const void* gu, void* out, void* stream) {
    tkv::clear_error();
    if (n_rows < 0 || inter < 1) return tkv::set_error(TKV_EINVAL, "tkv_swiglu: n_rows %d, inter %d", n_rows, inter);
    if (n_rows == 0) return TKV_OK;
    if (!gu || !out) return tkv::set_error(TKV_EINVAL, "tkv_swiglu: NULL pointer");
    const bool vec = inter % 8 == 0 && aligned16(gu) && aligned16(out);
    const int64_t n = static_cast<int64_t>(n_rows) * inter / (vec ? 8 : 1);
    const int64_t grid = (n + kThreads - 1) / kThreads;
    if (grid > kMaxGrid) return tkv::set_error(TKV_EINVAL, "tkv_swiglu: %d rows are too many", n_rows);
    const auto kernel = vec ? swiglu<true> : swiglu<false>;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, static_cast<hipStream_t>(stream), n,
                       static_cast<int64_t>(inter), static_cast<const uint16_t*>(gu), static_cast<uint16_t*>(out));
    return launched("tkv_swiglu");
}
