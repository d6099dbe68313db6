// The colour network's float32 form on the bfloat16 matrix cores.
//
// A float32 value is the exact sum of three bfloat16 values (planes hi, mid,
// lo: 8 bits of significand each, see store_planes), so a product of two
// float32 values is the sum of nine bfloat16 products, each exact in the
// matrix core's float32 accumulation.  Six of them are taken, hi*hi, hi*mid,
// mid*hi, mid*mid, hi*lo and lo*hi; the three left out are below 2^-26 of the
// product, a quarter of a float32 rounding.  Six K = 16 bfloat16 instructions
// replace eight K = 2 float32 ones of twice their duration: 2.7 times the
// rate, and 48 roundings of an accumulator over a 128-wide layer instead of
// 64.
#pragma once

#include "mlp_mfma.hpp"

namespace {

// The three planes of eight float32 values, in operand order.
struct Split8 {
    bf16x8 p[3];
};

template <typename V>
__device__ __forceinline__ Split8 split8(const V& v, int first) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    u32x4 w[3];
    #pragma unroll
    for (int e = 0; e < 4; ++e) {
        f32x2 x = {v[first + 2 * e], v[first + 2 * e + 1]};
        #pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
            w[p][e] = b;
            if (p < 2) {
                x[0] -= __uint_as_float(b << 16);
                x[1] -= __uint_as_float(b & 0xFFFF0000u);
            }
        }
    }
    Split8 s;
    #pragma unroll
    for (int p = 0; p < 3; ++p) s.p[p] = __builtin_bit_cast(bf16x8, w[p]);
    return s;
}

// acc[t] += A_t * B over kSteps K steps for the NT tiles t, the planes of A
// in LDS (plane stride kPlane fragments, tile stride kTile, one K step per 64
// fragments) and those of B from operand(step).  Each step takes A's planes
// from the smallest: lo with B's hi; mid with mid, hi; hi with lo, mid, hi.
// The NT fragments of the next plane are read from LDS while this one's
// instructions run (the order is pinned with scheduling-group barriers: the
// compiler would otherwise hoist every read to the front).
template <int NT, int kSteps, int kPlane, int kTile, typename Op>
__device__ __forceinline__ void split_chain(const bf16x8* w, int lane, f32x16 acc[NT], Op operand) {
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 cur[NT];
    #pragma unroll
    for (int t = 0; t < NT; ++t) cur[t] = w[2 * kPlane + t * kTile + lane];
    #pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        const Split8 x = operand(st);
        #pragma unroll
        for (int a = 2; a >= 0; --a) {
            bf16x8 nxt[NT];
            const int an = a > 0 ? a - 1 : 2, sn = a > 0 ? st : st + 1;
            if (sn < kSteps) {
                #pragma unroll
                for (int t = 0; t < NT; ++t) nxt[t] = w[an * kPlane + t * kTile + sn * 64 + lane];
            }
            #pragma unroll
            for (int b = 2 - a; b >= 0; --b)
                #pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = mma_bf16(cur[t], x.p[b], acc[t]);
            if (sn < kSteps) {
                #pragma unroll
                for (int t = 0; t < NT; ++t) cur[t] = nxt[t];
            }
        }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
    #pragma unroll
    for (int st = 0; st < kSteps; ++st) {
        __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 2 * NT, 0);
        if (st + 1 < kSteps) __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 3 * NT, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------
// forward: one wavefront per 32 samples, eight wavefronts per workgroup (two
// per SIMD, so that one wavefront's splits and loads run beside the other's
// matrix instructions), the planes of W1 and W2 in LDS.
// ---------------------------------------------------------------------------
template <int KX>
__global__ __launch_bounds__(512, 2) void mlp_fwd_split_kernel(MlpArgs a0, PosArgs pa) {
    using L = NetLayout<KX>;
    constexpr int kS1 = L::kS1;
    constexpr int kW1 = 4 * kS1 * 64;      // fragments of one plane of W1
    constexpr int kW2 = kW2PackBF16 / 8;   // and of W2
    __shared__ bf16x8 sW2[3 * kW2];
    __shared__ bf16x8 sW1[3 * kW1];
    __shared__ __attribute__((aligned(16))) float sB2[kH];
    __shared__ __attribute__((aligned(16))) float sW3[3 * kH];
    const int64_t n = *a0.n_kept < a0.cap ? *a0.n_kept : a0.cap;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // consecutive tiles go to one workgroup (a ray's samples share its
    // first-layer row in one L2), unless there are no more tiles than
    // wavefronts: then they are dealt over the workgroups first
    const bool few = n <= static_cast<int64_t>(gridDim.x) * 8 * 32;
    const int64_t first = few ? static_cast<int64_t>(wave) * gridDim.x + blockIdx.x
                              : static_cast<int64_t>(blockIdx.x) * 8 + wave;
    if ((few ? blockIdx.x : blockIdx.x * 8LL) * 32 >= n) return;   // no tile for the whole workgroup
    {
        Frags<512, 3 * kW2> f2;
        Frags<512, 3 * kW1> f1;
        f2.load(reinterpret_cast<const bf16x8*>(a0.w2pb));
        f1.load(reinterpret_cast<const bf16x8*>(a0.w1pb));
        const int t = static_cast<int>(threadIdx.x);
        const float v = t < 3 * kH ? a0.w3[t] : a0.b2[t - 3 * kH];
        f2.store(sW2);
        f1.store(sW1);
        if (t < 3 * kH) sW3[t] = v;
        else sB2[t - 3 * kH] = v;
    }
    __syncthreads();
    const float b3[3] = {a0.b3[0], a0.b3[1], a0.b3[2]};
    const int m = lane & 31, h = lane >> 5;
    for (int64_t tile = first; tile * 32 < n; tile += static_cast<int64_t>(gridDim.x) * 8) {
        // the lane's index into the operands, hidden from the optimiser: the
        // operands do not change, and it would move their reads out of the
        // loop into hundreds of registers
        int ln = lane, h4 = 4 * h;
        asm volatile("" : "+v"(ln), "+v"(h4));
        const int64_t s = tile * 32 + m;
        const bool ok = s < n;
        const int64_t sc = ok ? s : n - 1;
        const int r = a0.sample_ray[sc];
        float xs[L::kS];
        sample_inputs<KX>(pa, a0.feat, sc, r, xs);
        f32x16 h1[4];
        load_base(a0.base, r, h, h1);
        split_chain<4, kS1, kW1, kS1 * 64>(sW1, ln, h1, [&](int st) {
            float v[8];   // this lane half's inputs 16st + 8h .. + 7 (zero beyond kS)
            #pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k0 = 16 * st + e, k1 = k0 + 8;
                const float v0 = k0 < L::kS ? xs[k0 < L::kS ? k0 : 0] : 0.0f;
                const float v1 = k1 < L::kS ? xs[k1 < L::kS ? k1 : 0] : 0.0f;
                v[e] = h ? v1 : v0;
            }
            return split8(v, 0);
        });
        f32x16 z2[4];
        #pragma unroll
        for (int mt = 0; mt < 4; ++mt)
            #pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 b = *reinterpret_cast<const float4*>(sB2 + 32 * mt + 8 * q + h4);
                z2[mt][4 * q] = b.x;
                z2[mt][4 * q + 1] = b.y;
                z2[mt][4 * q + 2] = b.z;
                z2[mt][4 * q + 3] = b.w;
            }
        split_chain<4, 8, kW2, 8 * 64>(sW2, ln, z2, [&](int st) {
            float v[8];
            #pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = fmaxf(h1[st >> 1][8 * (st & 1) + e], 0.0f);
            return split8(v, 0);
        });
        // layer 3 in float32 on the vector units: W3 from LDS, the same
        // address in every lane of a half
        float z3[3] = {0.0f, 0.0f, 0.0f};
        #pragma unroll
        for (int mt = 0; mt < 4; ++mt)
            #pragma unroll
            for (int q = 0; q < 4; ++q)
                #pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float4 w = *reinterpret_cast<const float4*>(sW3 + c * kH + 32 * mt + 8 * q + h4);
                    z3[c] += w.x * fmaxf(z2[mt][4 * q], 0.0f);
                    z3[c] += w.y * fmaxf(z2[mt][4 * q + 1], 0.0f);
                    z3[c] += w.z * fmaxf(z2[mt][4 * q + 2], 0.0f);
                    z3[c] += w.w * fmaxf(z2[mt][4 * q + 3], 0.0f);
                }
        float col[3];
        #pragma unroll
        for (int c = 0; c < 3; ++c) {
            z3[c] += __shfl_xor(z3[c], 32, 64);
            col[c] = 1.0f / (1.0f + expf(-(z3[c] + b3[c])));
        }
        if (ok && h == 0) reinterpret_cast<float4*>(a0.col)[s] = make_float4(col[0], col[1], col[2], 0.0f);
    }
}

// kx: frequencies of the encoded position in the input (0 or kMaxKX).
// The bfloat16 forward (under 168 registers) fits three wavefronts per SIMD:
// three workgroups per compute unit (2 -> 3: 25.7 -> 23.9 us per step at the
// full configuration); the float32 one, two.
inline void launch_mlp_fwd(const MlpArgs& a, const PosArgs& pa, int kx, int cus, hipStream_t s) {
    if (a.bf16 && kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_FWD, mlp_fwd_bf16_kernel<kMaxKX>, dim3(cus * 3), dim3(256), 0, s, a, pa);
    else if (a.bf16) DVGO_LAUNCH(K_MLP_FWD, mlp_fwd_bf16_kernel<0>, dim3(cus * 3), dim3(256), 0, s, a, pa);
    else if (kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_FWD, mlp_fwd_split_kernel<kMaxKX>, dim3(cus), dim3(512), 0, s, a, pa);
    else DVGO_LAUNCH(K_MLP_FWD, mlp_fwd_split_kernel<0>, dim3(cus), dim3(512), 0, s, a, pa);
}
inline void launch_mlp_bwd(const MlpArgs& a, const PosArgs& pa, int kx, int blocks, hipStream_t s) {
    if (a.bf16 && kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_bf16_kernel<kMaxKX>, dim3(blocks), dim3(512), 0, s, a, pa);
    else if (a.bf16) DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_bf16_kernel<0>, dim3(blocks), dim3(512), 0, s, a, pa);
    else if (kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_f32_kernel<kMaxKX>, dim3(blocks), dim3(256), 0, s, a, pa);
    else DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_f32_kernel<0>, dim3(blocks), dim3(256), 0, s, a, pa);
}

}  // namespace
