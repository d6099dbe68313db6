// The colour network's float32 form on the bfloat16 matrix cores.
//
// A float32 value is the exact sum of three bfloat16 values (planes hi, mid,
// lo: 8 bits of significand each, see store_planes; the splitting of a wide
// float into narrow ones goes back to Dekker, 1971), so a product of two
// float32 values is the sum of nine bfloat16 products, each exact in the
// matrix core's float32 accumulation.  Six of them are taken, hi*hi, hi*mid,
// mid*hi, mid*mid, hi*lo and lo*hi; the three left out are at most 2^-24 of the
// product, half a unit in float32's last place, and 2^-27.4 rms.  Six K = 16
// bfloat16 instructions replace eight K = 2 float32 ones of twice their
// duration: 2.7 times the rate, and 48 roundings of an accumulator over a
// 128-wide layer instead of 64.
//
// Range: a plane below 2^-126, the smallest normal bfloat16, can count as zero,
// so operands below about 2^-109 err by up to 2^-126 (float32 holds those down
// to 2^-149: gradients of samples that hardly any light reaches).  Scaling the
// gradients up would move that limit at the expense of the other one: a weight
// gradient of the largest float32 features would overflow.  Above the largest
// bfloat16 the high plane is infinite and the others are not numbers, so such an
// operand, or an infinity, makes every sum that it enters NaN.  The forward lets
// a NaN through its ReLUs, and a sample whose logits are not finite is evaluated
// by the plain float32 chain instead (plain_sample).  The adjoint's operands are
// h1 and the inputs, which the forward has checked in this way, and gradients:
// with dL/dc below 2^64 and weights below 2^20 those stay below 2^112.  Where
// either is not so, or a sample's logits were not finite, the adjoint takes the
// plain chain for every sample (plain_adjoint).
#pragma once

#include <type_traits>

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

// The six products (planes of A and B), smallest first.
constexpr int kTermA[6] = {2, 0, 1, 1, 0, 0};
constexpr int kTermB[6] = {0, 2, 1, 0, 1, 0};

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

// The ReLU branches of a sample for the adjoint, one bit per hidden unit:
// word h*4 + mt of a sample holds the units of registers 0..15 of tile mt in
// lane half h (register i at bit 15 - i), layer 1 in the high and layer 2 in
// the low 16 bits.
//
// A gradient jumps by a sample's whole share where a unit changes its branch,
// and near zero the pre-activation's rounding decides that.  Such branches are
// taken from the plain float32 chain of fused multiply-adds, in input order
// (a float32 matrix instruction's own order and rounding): a sample with a unit
// within 2^-20 of zero, relative to the largest of its lane, has the chain
// evaluated, one sample in about two thousand; any other unit has the split
// chain's sign.  The two chains differ by about 2^-22 of a layer's rms, so the
// distance is ample where a unit's terms are of its layer's size; it is no
// bound for terms that all cancel to far below theirs.  A unit at exactly zero
// counts as near; one without weights and bias is not at zero (kDeadBias).
__device__ __forceinline__ uint32_t add_live(uint32_t bits, const f32x16& z, float* lo, float* hi) {
    #pragma unroll
    for (int i = 0; i < 16; i += 2) {
        *lo = fminf(fminf(*lo, fabsf(z[i])), fabsf(z[i + 1]));
        *hi = fmaxf(fmaxf(*hi, fabsf(z[i])), fabsf(z[i + 1]));
    }
    // the sign of 0 - z (set only for z > 0), shifted in from the right
    #pragma unroll
    for (int i = 0; i < 16; ++i)
        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(0.0f - z[i]), 31);
    return bits;
}

// The units of a tile whose bit m (row m of the tile) is set in t, as the 16
// register bits of lane half h.
__device__ __forceinline__ uint32_t half_bits(uint32_t t, int h) {
    t >>= 4 * h;
    const uint32_t b = (t & 0xFu) | (t >> 4 & 0xF0u) | (t >> 8 & 0xF00u) | (t >> 12 & 0xF000u);
    return __builtin_bitreverse32(b) >> 16;
}

// The branches and the colour of the sample of column ms by the plain chain,
// one unit per lane and pass; scratch: 128 floats of LDS.  The whole wavefront
// takes part; the results go to the sample's two lanes.
template <int KX>
__device__ __forceinline__ void plain_sample(const MlpArgs& a, const float xs[NetLayout<KX>::kS], int r, int ms,
                                             int lane, float* scratch, uint32_t live[4], float col[3]) {
    using L = NetLayout<KX>;
    const int m = lane & 31;
    const int rs = __builtin_amdgcn_readlane(r, ms);
    const float4* w1p = reinterpret_cast<const float4*>(a.w1p);
    const float4* w2p = reinterpret_cast<const float4*>(a.w2p);
    uint32_t tile1[4], tile2[4];
    #pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int mt = 2 * p + (lane >> 5);
        float acc = a.base[static_cast<int64_t>(rs) * kH + 32 * mt + m];
        #pragma unroll
        for (int q = 0; q < L::kQ1; ++q) {
            const float4 e = w1p[(mt * L::kQ1 + q) * 64 + m], o = w1p[(mt * L::kQ1 + q) * 64 + 32 + m];
            #pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = 2 * (4 * q + u);
                auto x = [&](int i) {
                    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(xs[i < L::kS ? i : 0]), ms));
                };
                if (k < L::kS) acc = fmaf(e[u], x(k), acc);
                if (k + 1 < L::kS) acc = fmaf(o[u], x(k + 1), acc);
            }
        }
        const uint64_t b = __ballot(acc > 0.0f);
        tile1[2 * p] = static_cast<uint32_t>(b);
        tile1[2 * p + 1] = static_cast<uint32_t>(b >> 32);
        scratch[32 * mt + m] = fmaxf(acc, 0.0f);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float z3[3] = {0.0f, 0.0f, 0.0f};
    #pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int mt = 2 * p + (lane >> 5);
        float acc = a.b2[32 * mt + m];
        #pragma unroll 4
        for (int q = 0; q < 16; ++q) {
            const float4 e = w2p[(mt * 16 + q) * 64 + m], o = w2p[(mt * 16 + q) * 64 + 32 + m];
            const float* hq = scratch + 32 * (q >> 2) + 8 * (q & 3);
            #pragma unroll
            for (int u = 0; u < 4; ++u) acc = fmaf(o[u], hq[4 + u], fmaf(e[u], hq[u], acc));
        }
        const uint64_t b = __ballot(acc > 0.0f);
        tile2[2 * p] = static_cast<uint32_t>(b);
        tile2[2 * p + 1] = static_cast<uint32_t>(b >> 32);
        #pragma unroll
        for (int c = 0; c < 3; ++c) z3[c] += a.w3[c * kH + 32 * mt + m] * fmaxf(acc, 0.0f);
    }
    __builtin_amdgcn_wave_barrier();
    #pragma unroll
    for (int c = 0; c < 3; ++c) z3[c] = wave_total(z3[c]);
    if (m == ms) {
        #pragma unroll
        for (int mt = 0; mt < 4; ++mt)
            live[mt] = half_bits(tile1[mt], lane >> 5) << 16 | half_bits(tile2[mt], lane >> 5);
        #pragma unroll
        for (int c = 0; c < 3; ++c) col[c] = 1.0f / (1.0f + expf(-(z3[c] + a.b3[c])));
    }
}

// ReLU that lets a NaN through (a NaN of the split sums is an operand out of
// the planes' range, of which the logits have to tell).
__device__ __forceinline__ float relu_nan(float z) { return __builtin_elementwise_maximum(z, 0.0f); }

// ---------------------------------------------------------------------------
// forward: one wavefront per 32 samples, eight wavefronts per workgroup (two
// per SIMD, so that one wavefront's splits and loads run beside the other's
// matrix instructions), the planes of W1 and W2 in LDS.  Bound by the matrix
// cores: 216 instructions of 32 cycles per 32 samples are 38 us for the full
// configuration's 390k samples; 59 us measured (126 us with float32 matrix
// instructions), 77 us with the branches for the adjoint (kLive).
// ---------------------------------------------------------------------------
template <int KX, bool kLive>
__global__ __launch_bounds__(512, 2) void mlp_fwd_split_kernel(MlpArgs a0, PosArgs pa) {
    using L = NetLayout<KX>;
    constexpr int kS1 = L::kS1;
    constexpr int kW1 = 4 * kS1 * 64;      // fragments of one plane of W1
    constexpr int kW2 = kW2PackBF16 / 8;   // and of W2
    __shared__ bf16x8 sW2[3 * kW2];
    __shared__ bf16x8 sW1[3 * kW1];
    __shared__ __attribute__((aligned(16))) float sB2[kH];
    __shared__ __attribute__((aligned(16))) float sW3[3 * kH];
    __shared__ __attribute__((aligned(16))) float sPlain[8][kH];
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
        if (kLive && blockIdx.x == 0) {   // weights of 2^20 and more, for the adjoint
            bool big = t < 3 * kH && !(fabsf(v) < 0x1p20f);
            auto any = [&](const bf16x8& w) {
                const i16x8 b = __builtin_bit_cast(i16x8, w);
                #pragma unroll
                for (int e = 0; e < 8; ++e) big |= (b[e] & 0x7FFF) >= 0x4980;
            };
            static_assert(kW2 % 512 == 0, "the first plane in whole rounds");
            #pragma unroll
            for (int u = 0; u < kW2 / 512; ++u) any(f2.t[u]);
            #pragma unroll
            for (int u = 0; u < (kW1 + 511) / 512; ++u)   // (and some of the smaller planes')
                if (u * 512 + t < 3 * kW1) any(f1.t[u]);
            if (__any(big) && lane == 0) *a0.wide = 1;
        }
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
        uint32_t live[4] = {0u, 0u, 0u, 0u};
        float lo1 = INFINITY, hi1 = 0.0f, lo2 = INFINITY, hi2 = 0.0f;   // smallest and largest |z| of the lane
        if constexpr (kLive) {
            #pragma unroll
            for (int mt = 0; mt < 4; ++mt) live[mt] = add_live(0u, h1[mt], &lo1, &hi1);
        }
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
            for (int e = 0; e < 8; ++e) v[e] = relu_nan(h1[st >> 1][8 * (st & 1) + e]);
            return split8(v, 0);
        });
        if constexpr (kLive) {
            #pragma unroll
            for (int mt = 0; mt < 4; ++mt) live[mt] = add_live(live[mt], z2[mt], &lo2, &hi2);
        }
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
                    z3[c] += w.x * relu_nan(z2[mt][4 * q]);
                    z3[c] += w.y * relu_nan(z2[mt][4 * q + 1]);
                    z3[c] += w.z * relu_nan(z2[mt][4 * q + 2]);
                    z3[c] += w.w * relu_nan(z2[mt][4 * q + 3]);
                }
        float col[3];
        #pragma unroll
        for (int c = 0; c < 3; ++c) {
            z3[c] += __shfl_xor(z3[c], 32, 64);
            col[c] = 1.0f / (1.0f + expf(-(z3[c] + b3[c])));
        }
        // out of the planes' range, or infinite or NaN in float32 as well
        const bool bad = ok && !(fabsf(z3[0]) + fabsf(z3[1]) + fabsf(z3[2]) < INFINITY);
        bool again = bad;
        if constexpr (kLive) {
            // (all 64 units at zero: no active input and no bias, zero in either chain)
            again |= ok && ((lo1 <= hi1 * 0x1p-20f && hi1 > 0.0f) || (lo2 <= hi2 * 0x1p-20f && hi2 > 0.0f));
        }
        if (const uint64_t mask = __ballot(again)) {
            float xa[L::kS], ca[3];   // (the inputs a second time: held until here, they spilled)
            int ra = r;
            asm volatile("" : "+v"(ra));
            sample_inputs<KX>(pa, refresh(a0).feat, sc, ra, xa);
            for (uint32_t todo = static_cast<uint32_t>(mask) | static_cast<uint32_t>(mask >> 32); todo; todo &= todo - 1)
                plain_sample<KX>(refresh(a0), xa, ra, __builtin_ctz(todo), lane, sPlain[wave], live, ca);
            #pragma unroll
            for (int c = 0; c < 3; ++c) col[c] = bad ? ca[c] : col[c];
            if (kLive && __any(bad) && lane == 0) *a0.wide = 1;
        }
        if (ok && h == 0) reinterpret_cast<float4*>(a0.col)[s] = make_float4(col[0], col[1], col[2], 0.0f);
        if (kLive && ok) reinterpret_cast<uint4*>(a0.live)[2 * s + h] = make_uint4(live[0], live[1], live[2], live[3]);
    }
}

// ---------------------------------------------------------------------------
// adjoint: weights stationary.  One workgroup of four wavefronts per compute
// unit, one wavefront per SIMD with the SIMD's whole register file.  Wavefront
// w owns features 32w .. 32w + 31 of every layer: it holds the planes of its
// rows of W2, then of W2^T, and its rows of every weight gradient in registers;
// the samples pass through in blocks of 64 (two column tiles), their
// activations exchanged through LDS as planes of [sample][feature] rows.  (The
// planes of W2 and W2^T alone are 192 KB, more than the LDS; this way an LDS
// byte read feeds 64 samples' worth of one wavefront's 32 rows, and the LDS
// takes half the time of the matrix instructions.)  One register set serves
// both matrices, refilled from the L2 in phases that do not use it: holding
// both spilled, and a spill's reload waits for every load before it.
//
// A block takes about 29,000 cycles, 11,900 of them matrix instructions; the
// rest is the vector work between two barriers that nothing overlaps (splits,
// head, dW3) and first loads.  387k samples: 334 us, about 750 with float32
// matrix instructions; 348 before the weight gradients' operands were read
// ahead and the head's weights once for both column tiles (with encoded
// positions 440 -> 415, 4096 rays in 128^3 145 -> 141).
// ---------------------------------------------------------------------------
// One lane's 16 values of its tile (accumulator order) as planes into its
// sample's row: `at` is the address of its first unit, the second is 2 further.
__device__ __forceinline__ void stage_tile(uint32_t at, const f32x16& v) {
    #pragma unroll
    for (int g = 0; g < 2; ++g) {
        const Split8 x = split8(v, 8 * g);
        #pragma unroll
        for (int p = 0; p < 3; ++p) lds_put((g ? at ^ 32u : at) + p * kPlaneB, x.p[p]);
    }
}

// The adjoint by plain float32 multiply-adds, for calls whose values may leave
// the planes' range (MlpArgs::wide): a sample at a time, thread (i, q) with the
// rows i and the columns of half q of both weight gradients in registers.  Not
// made to be fast (a run in which it is taken has diverged).  lds: 1024 floats.
template <int KX>
__device__ __forceinline__ void plain_adjoint(const MlpArgs& a, const PosArgs& pa, int64_t n, float* lds) {
    using L = NetLayout<KX>;
    constexpr int kCols = L::kIn + 1, kPer = (kCols + 1) / 2;   // columns of x' = [inputs, PE(d), 1]
    float *sX = lds, *sH = lds + 128, *sD2 = lds + 256, *sD1 = lds + 384, *sZ = lds + 512;
    static_assert(2 * kPer <= 128, "x' fits its row");
    const int t = static_cast<int>(threadIdx.x), i = t & (kH - 1), q = t >> 7;
    float dW2[kH / 2], dW1[kPer], dW3[3] = {0.0f, 0.0f, 0.0f}, db2 = 0.0f, db3[3] = {0.0f, 0.0f, 0.0f};
    #pragma unroll
    for (int j = 0; j < kH / 2; ++j) dW2[j] = 0.0f;
    #pragma unroll
    for (int j = 0; j < kPer; ++j) dW1[j] = 0.0f;
    if (t < 128) sX[t] = 0.0f;
    for (int64_t s = blockIdx.x; s < n; s += gridDim.x) {
        __syncthreads();   // the last sample's rows read
        const int r = a.sample_ray[s];
        if (t < kC) {
            sX[t] = a.feat[s * kC + t];
        } else if (t < L::kS) {   // as sample_encode
            float o[3], d[3], x[3];
            for (int c = 0; c < 3; ++c) {
                o[c] = pa.rays_o[3 * r + c];
                d[c] = pa.rays_d[3 * r + c];
            }
            const float tk = dvgo_dev::recipe_tk(pa.t_near[r], pa.jitter ? pa.jitter[r] : 0.0f, pa.sample_k[s], pa.step);
            dvgo_dev::recipe_x(o, d, tk, x);
            const int e = t - kC, c = e % 3, f = (e - 3) / 6;   // u, then three sines and three cosines per frequency
            const float u = ((c == 0 ? x[0] : c == 1 ? x[1] : x[2]) - (c == 0 ? pa.pe_c[0] : c == 1 ? pa.pe_c[1] : pa.pe_c[2])) *
                            (c == 0 ? pa.pe_ih[0] : c == 1 ? pa.pe_ih[1] : pa.pe_ih[2]);
            float sv, cv;
            dvgo_dev::pe_sincos(u * static_cast<float>(1 << (e < 3 ? 0 : f)), &sv, &cv);
            sX[t] = e < 3 ? u : (e - 3) % 6 < 3 ? sv : cv;
        } else if (t < kCols) {
            sX[t] = a.pe[static_cast<int64_t>(r) * 32 + t - L::kS];
        }
        __syncthreads();
        float z1 = a.base[static_cast<int64_t>(r) * kH + i];
        for (int k = 0; k < L::kS; ++k) z1 = fmaf(a.w1[i * L::kIn + k], sX[k], z1);
        if (q == 0) sH[i] = fmaxf(z1, 0.0f);
        __syncthreads();
        float z2 = a.b2[i];
        for (int g = 0; g < kH; g += 8)   // the chain's order: see plain_sample
            for (int u = 0; u < 4; ++u) {
                z2 = fmaf(a.w2[i * kH + g + u], sH[g + u], z2);
                z2 = fmaf(a.w2[i * kH + g + 4 + u], sH[g + 4 + u], z2);
            }
        const float h2 = fmaxf(z2, 0.0f);
        float w3[3], p[3];
        #pragma unroll
        for (int c = 0; c < 3; ++c) {
            w3[c] = a.w3[c * kH + i];
            p[c] = wave_total(w3[c] * h2);
            if ((t & 63) == 0) sZ[4 * (t >> 6) + c] = p[c];
        }
        __syncthreads();
        const float4 dc = reinterpret_cast<const float4*>(a.col)[s];
        const float g[3] = {dc.x, dc.y, dc.z};
        float dz3[3];
        #pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float cv = 1.0f / (1.0f + expf(-(sZ[c] + sZ[4 + c] + a.b3[c])));
            dz3[c] = g[c] * cv * (1.0f - cv);
            db3[c] += dz3[c];
            dW3[c] += dz3[c] * h2;
        }
        const float dz2 = z2 > 0.0f ? w3[0] * dz3[0] + w3[1] * dz3[1] + w3[2] * dz3[2] : 0.0f;
        db2 += dz2;
        if (q == 0) sD2[i] = dz2;
        __syncthreads();
        float dh = 0.0f;
        for (int k = 0; k < kH; ++k) dh = fmaf(a.w2[k * kH + i], sD2[k], dh);
        const float dz1 = z1 > 0.0f ? dh : 0.0f;
        if (q == 0) sD1[i] = dz1;
        __syncthreads();
        #pragma unroll
        for (int j = 0; j < kH / 2; ++j) dW2[j] = fmaf(dz2, sH[kH / 2 * q + j], dW2[j]);
        #pragma unroll
        for (int j = 0; j < kPer; ++j) dW1[j] = fmaf(dz1, sX[kPer * q + j], dW1[j]);
        // the record: 16 threads per feature channel, the head by a thread beyond
        const int2 cr = a.cell_rank[s];
        float4* rec = a.rec + (static_cast<int64_t>(a.cell_start[cr.x]) + cr.y) * 4;
        if (t < 16 * kC) {
            float v = 0.0f;
            for (int k = t & 15; k < kH; k += 16) v = fmaf(a.w1[k * L::kIn + (t >> 4)], sD1[k], v);
            #pragma unroll
            for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            if ((t & 15) == 0) reinterpret_cast<float*>(rec + 1)[t >> 4] = v;
        } else if (t == 16 * kC) {
            rec[0] = a.rec_head[s];
        }
    }
    float* out = a.partial + static_cast<int64_t>(blockIdx.x) * L::kPStride;
    #pragma unroll
    for (int j = 0; j < kH / 2; ++j) out[L::kOffW2 + i * kH + kH / 2 * q + j] = dW2[j];
    #pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int col = kPer * q + j;
        if (col < L::kIn) out[L::kOffW1 + i * L::kIn + col] = dW1[j];
        else if (col == L::kIn) out[L::kOffB1 + i] = dW1[j];
    }
    if (q == 0) {
        #pragma unroll
        for (int c = 0; c < 3; ++c) out[L::kOffW3 + c * kH + i] = dW3[c];
        out[L::kOffB2 + i] = db2;
    }
    if (t < 3) out[L::kOffB3 + t] = t == 0 ? db3[0] : t == 1 ? db3[1] : db3[2];
}

template <int KX>
__global__ __launch_bounds__(256, 1) void mlp_bwd_split_kernel(MlpArgs a0, PosArgs pa) {
    using L = NetLayout<KX>;
    constexpr int kS1 = L::kS1;
    constexpr int kXP = KX > 0 ? 112 : 80;      // pitch of an x' row
    constexpr int kGroups = (L::kIn + 1 + 7) / 8;   // 8-column groups of x' = [inputs, PE(d), 1]
    constexpr int kXTile = kSB * kXP;
    constexpr int kXF = 8 * kGroups + 4;        // pitch of the float32 x' rows (KX > 0)
    constexpr int kW1 = 4 * kS1 * 64, kW2 = kW2PackBF16 / 8;
    __shared__ __attribute__((aligned(256))) __bf16 sH[3 * kTile];   // h1, then (own columns) dL/dz1
    __shared__ __attribute__((aligned(256))) __bf16 sZ[3 * kTile];   // dL/dz2
    __shared__ __attribute__((aligned(256))) __bf16 sX[3 * kXTile];  // x'
    __shared__ __attribute__((aligned(16))) float sD[4][kSB][kC];    // the wavefronts' dL/dfeat
    __shared__ __attribute__((aligned(16))) float sL[4][kSB][4];     // the wavefronts' logits
    __shared__ __attribute__((aligned(16))) float sW3[3 * kH];
    __shared__ __attribute__((aligned(16))) float sB2[kH];
    static_assert(kSB * kXF * 4 <= static_cast<int>(sizeof(sZ)), "the float32 x' rows share sZ");
    float* sXF = reinterpret_cast<float*>(sZ);
    const int64_t n = *a0.n_kept < a0.cap ? *a0.n_kept : a0.cap;
    const int t = static_cast<int>(threadIdx.x);
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m = lane & 31, h = lane >> 5;
    if (*a0.wide != 0) {
        plain_adjoint<KX>(a0, pa, n, sXF);
        return;
    }
    f32x16 dW2[4], dW1[L::kXT];
    #pragma unroll
    for (int i = 0; i < 4; ++i) dW2[i] = zero_tile();
    #pragma unroll
    for (int i = 0; i < L::kXT; ++i) dW1[i] = zero_tile();
    // per lane, over its own samples: rows acc_row(., h) of the wavefront's tile
    f32x16 dW3[3], db2 = zero_tile();
    #pragma unroll
    for (int c = 0; c < 3; ++c) dW3[c] = zero_tile();
    float db3[3] = {0.0f, 0.0f, 0.0f};
    for (int i = t; i < 3 * kXTile / 8; i += 256) {   // columns past the last group stay zero
        bf16x8 z;
        #pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = static_cast<__bf16>(0.0f);
        *reinterpret_cast<bf16x8*>(sX + 8 * i) = z;
    }
    for (int i = t; i < 3 * kH; i += 256) sW3[i] = a0.w3[i];
    if (t < kH) sB2[t] = a0.b2[t];
    const float b3[3] = {a0.b3[0], a0.b3[1], a0.b3[2]};
    __syncthreads();
    const int xrow = t >> 2, xq = t & 3;   // the x' row and first column group this thread stages
    // the wavefront's rows of W2 (layer 2) or W2^T (its adjoint): one register
    // set, refilled from the L2
    bf16x8 wf[8][3];
    auto load_w = [&](const uint16_t* w, int st) {
        const bf16x8* g = reinterpret_cast<const bf16x8*>(w) + wave * 512 + st * 64;
        #pragma unroll
        for (int p = 0; p < 3; ++p) wf[st][p] = (g + p * kW2)[lane];
    };
    // acc += wf * (rows of an activation tile): K step st + 1 is read from LDS
    // while step st's instructions run, and each step's fragments are replaced
    // by those of `next_w` once used (spread over the phase: 24 KB at once per
    // wavefront hold up the issue for 1500 cycles)
    auto chain = [&](uint32_t row, f32x16 acc[2], auto refill, const uint16_t* next_w) {
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 cur[2][3];
        auto rd = [&](int st, bf16x8 B[2][3]) {
            #pragma unroll
            for (int c = 0; c < 2; ++c)
                #pragma unroll
                for (int p = 0; p < 3; ++p)
                    B[c][p] = lds_get<bf16x8>((row ^ (32u * st)) + c * kColB + p * kPlaneB);
        };
        rd(0, cur);
        #pragma unroll
        for (int st = 0; st < 8; ++st) {
            bf16x8 nxt[2][3];
            if (st < 7) rd(st + 1, nxt);
            #pragma unroll
            for (int q = 0; q < 6; ++q)
                #pragma unroll
                for (int c = 0; c < 2; ++c) acc[c] = mma_bf16(wf[st][kTermA[q]], cur[c][kTermB[q]], acc[c]);
            if constexpr (refill.value) load_w(next_w, st);
            if (st < 7) {
                #pragma unroll
                for (int c = 0; c < 2; ++c)
                    #pragma unroll
                    for (int p = 0; p < 3; ++p) cur[c][p] = nxt[c][p];
            }
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
        #pragma unroll
        for (int st = 0; st < 8; ++st) {
            if (st < 7) __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 12, 0);
            if constexpr (refill.value) __builtin_amdgcn_sched_group_barrier(0x020, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // operand of a feature tile over samples 16st .. 16st + 15
    auto tr_unit = [&](uint32_t at, int st, int p) {
        const uint32_t off = st * (16 * kH * 2) + p * kPlaneB;
        return tr_pair(at + off, (at ^ 16u) + 4 * kH * 2 + off);
    };
    // A block's samples by a scalar base and a 32-bit lane offset (the last
    // block's missing samples read its last one).
    const int nblocks = static_cast<int>((n + kSB - 1) / kSB);
    auto last_of = [&](int blk) {
        const int64_t left = n - static_cast<int64_t>(blk) * kSB;
        return static_cast<int>(left < kSB ? left : kSB) - 1;
    };
    // the rays of the next block's samples (this lane's two columns, and this
    // thread's x' row), loaded a block ahead
    int r_n[2], xr_n;
    auto load_rays = [&](const MlpArgs& a, int blk) {
        const int* sr = a.sample_ray + static_cast<int64_t>(blk) * kSB;
        const int last = last_of(blk);
        #pragma unroll
        for (int c = 0; c < 2; ++c) r_n[c] = sr[min(32 * c + m, last)];
        xr_n = sr[min(xrow, last)];
    };
    // this thread's x' columns (KX == 0), loaded while the block before ends
    float4 xin[4];
    auto load_x = [&](const MlpArgs& a, int blk) {
        if constexpr (KX == 0) {
            // groups: f[0..7] | f[8..11], PE[0..3] | PE[4..11] | PE[12..19] | PE[20..26], 1
            const float* f = a.feat + static_cast<int64_t>(blk) * (kSB * kC) + min(xrow, last_of(blk)) * kC;
            const float* pe = a.pe + static_cast<int64_t>(xr_n) * 32;
            xin[0] = *reinterpret_cast<const float4*>(xq < 2 ? f + 8 * xq : pe + 8 * xq - 12);
            xin[1] = *reinterpret_cast<const float4*>(xq < 1 ? f + 4 : pe + 8 * xq - 8);
            xin[2] = *reinterpret_cast<const float4*>(pe + 20);
            xin[3] = *reinterpret_cast<const float4*>(pe + 24);
        }
    };
    if (static_cast<int>(blockIdx.x) < nblocks) {
        load_rays(a0, blockIdx.x);
        load_x(a0, blockIdx.x);
        #pragma unroll
        for (int st = 0; st < 8; ++st) load_w(a0.w2pb, st);
    }
    for (int blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        const MlpArgs a = refresh(a0);
        // this lane's LDS addresses (hidden from the optimiser, which would
        // otherwise keep every sum of them in a register of its own):
        // its sample's row, unit h; the unit it stages; the first of its two
        // transpose reads of feature tile nt (the second is 4 rows on, where
        // the unit permutation differs in its lowest bit)
        const int tG = lane >> 4, tt = lane & 15, trow = 8 * (tG >> 1) + (tt >> 2);
        const uint32_t tsub = trow * 256 + 8 * ((tt & 3) >> 1), tu = 2 * (tG & 1) + (tt & 1);
        uint32_t rowH = lds_addr(sH) + m * 256 + 16 * (h ^ unit_swz(m));
        uint32_t rowZ = lds_addr(sZ) + m * 256 + 16 * (h ^ unit_swz(m));
        uint32_t putH = rowH ^ (64u * wave), putZ = rowZ ^ (64u * wave);
        uint32_t trH = lds_addr(sH) + tsub + 16 * (tu ^ unit_swz(trow));
        uint32_t trZ = (lds_addr(sZ) + tsub + 16 * (tu ^ unit_swz(trow))) ^ (64u * wave);
        uint32_t colX = lds_addr(sX) + (m * kXP + 8 * h) * 2;
        uint32_t trX = lds_addr(sX) + (trow * kXP + 16 * (tG & 1) + 4 * (tt & 3)) * 2;
        uint32_t putX = lds_addr(sX) + xrow * kXP * 2;
        asm volatile("" : "+v"(rowH), "+v"(rowZ), "+v"(putH), "+v"(putZ), "+v"(trH), "+v"(trZ), "+v"(colX), "+v"(trX),
                     "+v"(putX));
        // the next block of this workgroup, or (the last time) this one again
        const int next = blk + static_cast<int>(gridDim.x) < nblocks ? blk + static_cast<int>(gridDim.x) : blk;
        const int64_t s0 = static_cast<int64_t>(blk) * kSB;
        const int last = last_of(blk);
        const int xi = min(xrow, last);   // this thread's x' and record sample
        // this block's loads, in the order of their use: the wavefront's rows
        // of the first layer's per-ray part, W1, inputs of the head and the
        // records; the next block's rays
        float4 base4[2][4];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float4* br = reinterpret_cast<const float4*>(a.base + static_cast<int64_t>(r_n[c]) * kH) + 8 * wave + h;
            #pragma unroll
            for (int q = 0; q < 4; ++q) base4[c][q] = br[2 * q];
        }
        bf16x8 w1f[kS1][3];
        #pragma unroll
        for (int st = 0; st < kS1; ++st)
            #pragma unroll
            for (int p = 0; p < 3; ++p)
                w1f[st][p] = (reinterpret_cast<const bf16x8*>(a.w1pb) + p * kW1 + (wave * kS1 + st) * 64)[lane];
        uint32_t live[2];
        float4 dc[2];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int i = min(32 * c + m, last);
            live[c] = (a.live + 8 * s0)[8 * i + 4 * h + wave];
            dc[c] = (reinterpret_cast<const float4*>(a.col) + s0)[i];
        }
        const int2 cr = (a.cell_rank + s0)[xi];
        const float4 rh = (a.rec_head + s0)[xi];
        const int xr = xr_n;
        load_rays(a, next);
        // ---- x' rows as planes
        auto put_x = [&](int col, const float v[8]) {
            const Split8 x = split8(v, 0);
            #pragma unroll
            for (int p = 0; p < 3; ++p) lds_put(putX + 2 * col + p * (2 * kXTile), x.p[p]);
        };
        if constexpr (KX == 0) {
            const float v[8] = {xin[0].x, xin[0].y, xin[0].z, xin[0].w, xin[1].x, xin[1].y, xin[1].z, xin[1].w};
            put_x(8 * xq, v);
            if (xq == 0) {
                const float vl[8] = {xin[2].x, xin[2].y, xin[2].z, xin[2].w, xin[3].x, xin[3].y, xin[3].z, xin[3].w};
                put_x(32, vl);
            }
        } else {
            // the four threads of a row evaluate the encoded position (thread
            // q frequency q, thread 3 also frequency 4) and copy the rest
            float* row = sXF + xrow * kXF;
            float x[3], u[3], o[3], d[3];
            #pragma unroll
            for (int i = 0; i < 3; ++i) {
                o[i] = pa.rays_o[3 * xr + i];
                d[i] = pa.rays_d[3 * xr + i];
            }
            const float tk = dvgo_dev::recipe_tk(pa.t_near[xr], pa.jitter ? pa.jitter[xr] : 0.0f,
                                                 (pa.sample_k + s0)[xi], pa.step);
            dvgo_dev::recipe_x(o, d, tk, x);
            #pragma unroll
            for (int i = 0; i < 3; ++i) u[i] = (x[i] - pa.pe_c[i]) * pa.pe_ih[i];
            const float* f = a.feat + s0 * kC + xi * kC;
            const float* pe = a.pe + static_cast<int64_t>(xr) * 32;
            // features by threads 0..2, the view encoding (32 values) by all
            if (xq < 3) *reinterpret_cast<float4*>(row + 4 * xq) = *reinterpret_cast<const float4*>(f + 4 * xq);
            const float4 e0 = *reinterpret_cast<const float4*>(pe + 8 * xq);
            const float4 e1 = *reinterpret_cast<const float4*>(pe + 8 * xq + 4);
            const float ev[8] = {e0.x, e0.y, e0.z, e0.w, e1.x, e1.y, e1.z, e1.w};
            #pragma unroll
            for (int e = 0; e < 8; ++e) row[L::kS + 8 * xq + e] = ev[e];
            if (xq == 0) {
                #pragma unroll
                for (int i = 0; i < 3; ++i) row[kC + i] = u[i];
            }
            for (int j = xq; j < KX; j += xq == 3 ? 1 : KX) {
                #pragma unroll
                for (int i = 0; i < 3; ++i) {
                    float sv, cv;
                    dvgo_dev::pe_sincos(u[i] * static_cast<float>(1 << j), &sv, &cv);
                    row[kC + 3 + 6 * j + i] = sv;
                    row[kC + 6 + 6 * j + i] = cv;
                }
            }
            __syncthreads();
            for (int g = xq; g < kGroups; g += 4) {
                const float4 u0 = *reinterpret_cast<const float4*>(row + 8 * g);
                const float4 u1 = *reinterpret_cast<const float4*>(row + 8 * g + 4);
                const float v[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
                put_x(8 * g, v);
            }
        }
        // the wavefront's rows of the per-ray first-layer part
        f32x16 h1[2];
        #pragma unroll
        for (int c = 0; c < 2; ++c)
            #pragma unroll
            for (int q = 0; q < 4; ++q) {
                h1[c][4 * q] = base4[c][q].x;
                h1[c][4 * q + 1] = base4[c][q].y;
                h1[c][4 * q + 2] = base4[c][q].z;
                h1[c][4 * q + 3] = base4[c][q].w;
            }
        __syncthreads();   // x' rows complete
        // ---- layer 1 (columns past the per-sample inputs meet zero weights)
        #pragma unroll
        for (int st = 0; st < kS1; ++st) {
            bf16x8 B[2][3];
            #pragma unroll
            for (int p = 0; p < 3; ++p)
                #pragma unroll
                for (int c = 0; c < 2; ++c)
                    B[c][p] = lds_get<bf16x8>(colX + (p * kXTile + 32 * c * kXP + 16 * st) * 2);
            #pragma unroll
            for (int q = 0; q < 6; ++q)
                #pragma unroll
                for (int c = 0; c < 2; ++c) h1[c] = mma_bf16(w1f[st][kTermA[q]], B[c][kTermB[q]], h1[c]);
        }
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            #pragma unroll
            for (int i = 0; i < 16; ++i) h1[c][i] = fmaxf(h1[c][i], 0.0f);
            stage_tile(putH + c * kColB, h1[c]);
        }
        f32x16 z2[2];
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 b = *reinterpret_cast<const float4*>(sB2 + 32 * wave + 8 * q + 4 * h);
            #pragma unroll
            for (int c = 0; c < 2; ++c) {
                z2[c][4 * q] = b.x;
                z2[c][4 * q + 1] = b.y;
                z2[c][4 * q + 2] = b.z;
                z2[c][4 * q + 3] = b.w;
            }
        }
        __syncthreads();   // h1 rows complete
        // ---- layer 2
        chain(rowH, z2, std::true_type{}, a.w2tpb);
        // operand of dL/dfeat
        bf16x8 w1t[2][3];
        #pragma unroll
        for (int g = 0; g < 2; ++g)
            #pragma unroll
            for (int p = 0; p < 3; ++p)
                w1t[g][p] = (reinterpret_cast<const bf16x8*>(a.w1tpb) + (p * 8 + 2 * wave + g) * 64)[lane];
        const int slot = a.cell_start[cr.x];
        // ---- head: the wavefront's share of the logits
        {
            float z3[2][3] = {{0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}};
            #pragma unroll
            for (int ch = 0; ch < 3; ++ch)
                #pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 w = *reinterpret_cast<const float4*>(sW3 + ch * kH + 32 * wave + 8 * q + 4 * h);
                    #pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        z3[c][ch] += w.x * fmaxf(z2[c][4 * q], 0.0f);
                        z3[c][ch] += w.y * fmaxf(z2[c][4 * q + 1], 0.0f);
                        z3[c][ch] += w.z * fmaxf(z2[c][4 * q + 2], 0.0f);
                        z3[c][ch] += w.w * fmaxf(z2[c][4 * q + 3], 0.0f);
                    }
                }
            #pragma unroll
            for (int c = 0; c < 2; ++c) {
                #pragma unroll
                for (int ch = 0; ch < 3; ++ch) z3[c][ch] += __shfl_xor(z3[c][ch], 32, 64);
                if (h == 0)
                    *reinterpret_cast<float4*>(sL[wave][32 * c + m]) = make_float4(z3[c][0], z3[c][1], z3[c][2], 0.0f);
            }
        }
        __syncthreads();   // logits complete
        // ---- dz3, dW3, db3, and dz2 = (W3^T dz3) * relu'(z2) into sZ
        float dz3[2][3];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            float z[3] = {b3[0], b3[1], b3[2]};
            #pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float4 v = *reinterpret_cast<const float4*>(sL[w][32 * c + m]);
                z[0] += v.x;
                z[1] += v.y;
                z[2] += v.z;
            }
            const float g[3] = {dc[c].x, dc[c].y, dc[c].z};
            #pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
                const float cv = 1.0f / (1.0f + expf(-z[ch]));
                dz3[c][ch] = 32 * c + m <= last ? g[ch] * cv * (1.0f - cv) : 0.0f;
                db3[ch] += dz3[c][ch];
            }
        }
        f32x16 dz[2];
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
            float4 w[3];
            #pragma unroll
            for (int ch = 0; ch < 3; ++ch)
                w[ch] = *reinterpret_cast<const float4*>(sW3 + ch * kH + 32 * wave + 8 * q + 4 * h);
            #pragma unroll
            for (int c = 0; c < 2; ++c)
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 4 * q + e;
                    const float h2 = fmaxf(z2[c][i], 0.0f);
                    #pragma unroll
                    for (int ch = 0; ch < 3; ++ch) dW3[ch][i] += dz3[c][ch] * h2;
                    const float dh = w[0][e] * dz3[c][0] + w[1][e] * dz3[c][1] + w[2][e] * dz3[c][2];
                    dz[c][i] = live[c] & (0x8000u >> i) ? dh : 0.0f;
                    db2[i] += dz[c][i];
                }
        }
        #pragma unroll
        for (int c = 0; c < 2; ++c) stage_tile(putZ + c * kColB, dz[c]);
        f32x16 d1[2] = {zero_tile(), zero_tile()};
        load_x(a, next);
        __syncthreads();   // dz2 rows complete
        // ---- dh1 = W2^T dz2, dz1 = dh1 * relu'(z1)
        chain(rowZ, d1, std::false_type{}, nullptr);
        Split8 dp[2][2];
        #pragma unroll
        for (int c = 0; c < 2; ++c) {
            #pragma unroll
            for (int i = 0; i < 16; ++i) d1[c][i] = live[c] & (0x80000000u >> i) ? d1[c][i] : 0.0f;
            #pragma unroll
            for (int g = 0; g < 2; ++g) dp[c][g] = split8(d1[c], 8 * g);
        }
        // ---- this wavefront's share of dL/dfeat = W1[:, :12]^T dz1 (K order
        // of the chain: the accumulator registers are the operand)
        {
            f32x16 df[2] = {zero_tile(), zero_tile()};
            #pragma unroll
            for (int g = 0; g < 2; ++g) {
                #pragma unroll
                for (int q = 0; q < 6; ++q)
                    #pragma unroll
                    for (int c = 0; c < 2; ++c) df[c] = mma_bf16(w1t[g][kTermA[q]], dp[c][g].p[kTermB[q]], df[c]);
            }
            // rows 0..11 of the tile: registers 0..3 are channels 4h .. 4h + 3,
            // registers 4..7 (half 0) channels 8..11
            #pragma unroll
            for (int c = 0; c < 2; ++c) {
                *reinterpret_cast<float4*>(&sD[wave][32 * c + m][4 * h]) =
                    make_float4(df[c][0], df[c][1], df[c][2], df[c][3]);
                if (h == 0)
                    *reinterpret_cast<float4*>(&sD[wave][32 * c + m][8]) =
                        make_float4(df[c][4], df[c][5], df[c][6], df[c][7]);
            }
        }
        // ---- dW2 rows 32w .. over the block's samples, the operands of two of
        // its tiles on their way from LDS while the two before are multiplied
        // (one wavefront per SIMD: nothing else covers the reads)
        {
            bf16x8 A[2][3], B[2][2][3];
            auto rd = [&](int k) {   // group k: K step k / 2, tiles 2 (k % 2) and the next
                #pragma unroll
                for (int p = 0; p < 3; ++p) {
                    if (k % 2 == 0) A[k / 2 % 2][p] = tr_unit(trZ, k / 2, p);
                    #pragma unroll
                    for (int c = 0; c < 2; ++c) B[k % 2][c][p] = tr_unit(trH ^ (64u * (2 * (k % 2) + c)), k / 2, p);
                }
            };
            __builtin_amdgcn_sched_barrier(0);
            rd(0);
            #pragma unroll
            for (int k = 0; k < 2 * kSB / 16; ++k) {
                if (k + 1 < 2 * kSB / 16) rd(k + 1);
                #pragma unroll
                for (int q = 0; q < 6; ++q)
                    #pragma unroll
                    for (int c = 0; c < 2; ++c)
                        dW2[2 * (k % 2) + c] = mma_bf16(A[k / 2 % 2][kTermA[q]], B[k % 2][c][kTermB[q]],
                                                        dW2[2 * (k % 2) + c]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();   // h1 rows read; dL/dfeat shares complete
        // dz1 into this wavefront's own columns of sH
        #pragma unroll
        for (int c = 0; c < 2; ++c)
            #pragma unroll
            for (int g = 0; g < 2; ++g)
                #pragma unroll
                for (int p = 0; p < 3; ++p)
                    lds_put((g ? putH ^ 32u : putH) + c * kColB + p * kPlaneB, dp[c][g].p[p]);
        // the sample's record, one 16-byte word per thread of its row
        {
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            #pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float4 u = *reinterpret_cast<const float4*>(&sD[w][xrow][xq > 0 ? 4 * (xq - 1) : 0]);
                v.x += u.x;
                v.y += u.y;
                v.z += u.z;
                v.w += u.w;
            }
            v.x = xq > 0 ? v.x : rh.x;
            v.y = xq > 0 ? v.y : rh.y;
            v.z = xq > 0 ? v.z : rh.z;
            v.w = xq > 0 ? v.w : rh.w;
            if (xrow <= last) a.rec[(static_cast<int64_t>(slot) + cr.y) * 4 + xq] = v;
        }
        // ---- dW1 rows 32w .. (column kIn: the bias); the wavefront reads
        // back its own dz1 rows, x' is everyone's
        {
            bf16x8 A[2][3], B[2][L::kXT][3];
            auto rd = [&](int st) {
                #pragma unroll
                for (int p = 0; p < 3; ++p) {
                    A[st % 2][p] = tr_unit(trH ^ (64u * wave), st, p);
                    #pragma unroll
                    for (int nt = 0; nt < L::kXT; ++nt) {
                        const uint32_t at = trX + (p * kXTile + 16 * st * kXP + 32 * nt) * 2;
                        B[st % 2][nt][p] = tr_pair(at, at + 4 * kXP * 2);
                    }
                }
            };
            __builtin_amdgcn_sched_barrier(0);
            rd(0);
            #pragma unroll
            for (int st = 0; st < kSB / 16; ++st) {
                if (st + 1 < kSB / 16) rd(st + 1);
                // W2 for the next block's layer 2
                load_w(a.w2pb, 2 * st);
                load_w(a.w2pb, 2 * st + 1);
                #pragma unroll
                for (int q = 0; q < 6; ++q)
                    #pragma unroll
                    for (int nt = 0; nt < L::kXT; ++nt)
                        dW1[nt] = mma_bf16(A[st % 2][kTermA[q]], B[st % 2][nt][kTermB[q]], dW1[nt]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();   // x', sD and sH read before the next block's staging
    }
    // ---- epilogue: this workgroup's partial of the flat gradient
    float* out = a0.partial + static_cast<int64_t>(blockIdx.x) * L::kPStride;
    #pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 32 * wave + acc_row(i, h);
        #pragma unroll
        for (int nt = 0; nt < 4; ++nt) out[L::kOffW2 + row * kH + 32 * nt + m] = dW2[nt][i];
        #pragma unroll
        for (int nt = 0; nt < L::kXT; ++nt) {
            const int col = 32 * nt + m;
            if (col < L::kIn) out[L::kOffW1 + row * L::kIn + col] = dW1[nt][i];
            else if (col == L::kIn) out[L::kOffB1 + row] = dW1[nt][i];
        }
        // sums over the 32 lanes (samples) of each half
        float v[4] = {dW3[0][i], dW3[1][i], dW3[2][i], db2[i]};
        #pragma unroll
        for (int c = 0; c < 4; ++c) {
            #pragma unroll
            for (int off = 16; off > 0; off >>= 1) v[c] += __shfl_xor(v[c], off, 64);
        }
        if (m < 3) out[L::kOffW3 + m * kH + row] = m == 0 ? v[0] : m == 1 ? v[1] : v[2];
        else if (m == 3) out[L::kOffB2 + row] = v[3];
    }
    #pragma unroll
    for (int c = 0; c < 3; ++c) {   // every lane of half 0 holds its own samples' sums
        #pragma unroll
        for (int off = 16; off > 0; off >>= 1) db3[c] += __shfl_xor(db3[c], off, 64);
    }
    if (t < 3) out[L::kOffB3 + t] = t == 0 ? db3[0] : t == 1 ? db3[1] : db3[2];
}

// kx: frequencies of the encoded position in the input (0 or kMaxKX).
// The bfloat16 forward (under 168 registers) fits three wavefronts per SIMD:
// three workgroups per compute unit (2 -> 3: 25.7 -> 23.9 us per step at the
// full configuration); the float32 one, two.
inline void launch_mlp_fwd(const MlpArgs& a, const PosArgs& pa, int kx, int cus, hipStream_t s) {
    if (a.bf16 && kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_FWD, mlp_fwd_bf16_kernel<kMaxKX>, dim3(cus * 3), dim3(256), 0, s, a, pa);
    else if (a.bf16) DVGO_LAUNCH(K_MLP_FWD, mlp_fwd_bf16_kernel<0>, dim3(cus * 3), dim3(256), 0, s, a, pa);
    else if (a.live && kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_FWD, (mlp_fwd_split_kernel<kMaxKX, true>), dim3(cus), dim3(512), 0, s, a, pa);
    else if (a.live) DVGO_LAUNCH(K_MLP_FWD, (mlp_fwd_split_kernel<0, true>), dim3(cus), dim3(512), 0, s, a, pa);
    else if (kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_FWD, (mlp_fwd_split_kernel<kMaxKX, false>), dim3(cus), dim3(512), 0, s, a, pa);
    else DVGO_LAUNCH(K_MLP_FWD, (mlp_fwd_split_kernel<0, false>), dim3(cus), dim3(512), 0, s, a, pa);
}
inline void launch_mlp_bwd(const MlpArgs& a, const PosArgs& pa, int kx, int blocks, hipStream_t s) {
    if (a.bf16 && kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_bf16_kernel<kMaxKX>, dim3(blocks), dim3(512), 0, s, a, pa);
    else if (a.bf16) DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_bf16_kernel<0>, dim3(blocks), dim3(512), 0, s, a, pa);
    else if (kx == kMaxKX)
        DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_split_kernel<kMaxKX>, dim3(blocks), dim3(256), 0, s, a, pa);
    else DVGO_LAUNCH(K_MLP_BWD, mlp_bwd_split_kernel<0>, dim3(blocks), dim3(256), 0, s, a, pa);
}

}  // namespace
