// Forward volume rendering of the fine stage and its adjoint (paper
// Eq. volume_rendering, Eq. fine_queries, Eq. post_activation,
// Eq. density_activation, Eq. photo_loss).
//
// One render call runs a short pipeline of kernels over the compact sample
// list written by dvgo_sample_rays; per-sample intermediates live in the
// caller's workspace:
//   prep     pack the network weights into matrix-core operand order;
//            per-ray view encoding PE(d) and the first layer's per-ray part
//   gather   trilinear density and feature interpolation per sample
//   mlp      colour network on the bfloat16 matrix cores (float32 operands
//            as three bfloat16 planes)
//   compose  per-ray front-to-back compositing with wavefront prefix scans
// and the backward pass adds
//   compose' walk each ray from its end (suffix scans from log_t_end)
//   mlp'     network adjoint, per-block weight-gradient partials
//   scatter  transpose of the trilinear interpolation: samples binned by
//            grid cell, a lane quad per vertex gathers its gradient (no
//            float atomics), the grids' Adam step fused in
//   reduce   deterministic sum of the per-block weight-gradient partials
#include "adam.hpp"
#include "binning.hpp"
#include "common.hpp"
#include "mlp_mfma.hpp"
#include "mlp_split.hpp"
#include "scan.hpp"

using dvgo::GridArgs;
using namespace dvgo_dev;

namespace {

constexpr int kMaxBwdBlocks = 256;

struct WsLayout {
    size_t base, pe, w1p, w2p, b2p, w1pb, w2pb, w2tpb, w3pb, w3tpb, w1tpb, raw, feat, col, partial, wide, cell_count,
        cell_start, scan_tmp, cell_rank, rec_head, rec, step_rgb, step_grad, step_logt, step_sqerr, live, total;
};

WsLayout ws_layout(int64_t B, int64_t cap, int64_t ncell) {
    WsLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = dvgo::align_up(off + bytes, 256);
        return o;
    };
    L.base = take(static_cast<size_t>(B) * kH * 4);
    L.pe = take(static_cast<size_t>(B) * 32 * 4);
    L.w1p = take(kW1PackF32Max * 4);
    L.w2p = take(kW2PackF32 * 4);
    L.b2p = take(kH * 4);
    L.w1pb = take(3 * kW1PackBF16Max * 2);   // the three planes of the float32 form
    L.w2pb = take(3 * kW2PackBF16 * 2);
    L.w2tpb = take(3 * kW2PackBF16 * 2);
    L.w3pb = take(kW3PackBF16 * 2);
    L.w3tpb = take(kW3TPackBF16 * 2);
    L.w1tpb = take(3 * kW1TPackBF16 * 2);
    L.raw = take(static_cast<size_t>(cap) * 4);
    L.feat = take(static_cast<size_t>(cap) * kC * 4);
    L.col = take(static_cast<size_t>(cap) * 4 * 4);
    L.partial = take(static_cast<size_t>(kMaxBwdBlocks) * kPStrideMax * 4);
    L.wide = take(4);
    L.cell_count = take(static_cast<size_t>(ncell + 1) * 4);
    L.cell_start = take(static_cast<size_t>(ncell + 1) * 4);
    L.scan_tmp = take(cell_scan_bytes(ncell + 1));
    L.cell_rank = take(static_cast<size_t>(cap) * 8);
    L.rec_head = take(static_cast<size_t>(cap) * 16);
    L.rec = take((static_cast<size_t>(cap) + 1) * 64);    // the last one zero (see vertex_sum)
    L.step_rgb = take(static_cast<size_t>(B) * 3 * 4);    // per-ray state of dvgo_train_step
    L.step_grad = take(static_cast<size_t>(B) * 3 * 4);
    L.step_logt = take(static_cast<size_t>(B) * 4);
    L.step_sqerr = take(static_cast<size_t>(B) * 4);
    L.live = take(static_cast<size_t>(cap) * 32);         // ReLU branches: the float32 network's adjoint only, so last
    L.total = off;
    return L;
}

// ---------------------------------------------------------------------------
// per-sample geometry (float32 recipe for t and x) and trilinear weights
// ---------------------------------------------------------------------------
struct SampleArgs {
    const float* rays_o;
    const float* rays_d;
    const float* jitter;
    const float* t_near;
    const int* sample_ray;
    const int* sample_k;
    float step;
};

__device__ __forceinline__ void sample_point(const SampleArgs& a, int r, int k, float x[3], float* t_out) {
    float o[3], d[3];
    for (int i = 0; i < 3; ++i) {
        o[i] = a.rays_o[3 * r + i];
        d[i] = a.rays_d[3 * r + i];
    }
    const float p = a.jitter ? a.jitter[r] : 0.0f;
    const float t = recipe_tk(a.t_near[r], p, k, a.step);
    recipe_x(o, d, t, x);
    if (t_out) *t_out = t;
}

struct Tri {
    int64_t base;   // linear vertex index of corner (0,0,0)
    int sx, sy;     // vertex strides of x and y (z stride 1)
    float w[8];     // corner c = (c>>2 &1, c>>1 &1, c &1)
};

__device__ __forceinline__ Tri trilinear(const GridArgs& g, const float x[3]) {
    int i0[3];
    float f[3];
    for (int i = 0; i < 3; ++i) {
        const float u = (x[i] - g.mn[i]) * g.scale[i];
        const float fl = fminf(fmaxf(floorf(u), 0.0f), static_cast<float>(g.n[i] - 2));
        i0[i] = static_cast<int>(fl);
        f[i] = fminf(fmaxf(u - fl, 0.0f), 1.0f);
    }
    Tri t;
    t.sy = g.n[2];
    t.sx = g.n[1] * g.n[2];
    t.base = (static_cast<int64_t>(i0[0]) * g.n[1] + i0[1]) * g.n[2] + i0[2];
    const float gx[2] = {1.0f - f[0], f[0]}, gy[2] = {1.0f - f[1], f[1]}, gz[2] = {1.0f - f[2], f[2]};
    for (int c = 0; c < 8; ++c) t.w[c] = gx[(c >> 2) & 1] * gy[(c >> 1) & 1] * gz[c & 1];
    return t;
}

// First corner of the point's cell and the position in the cell, as trilinear forms them.
__device__ __forceinline__ int64_t cell_base(const GridArgs& g, const float x[3], float f[3]) {
    int i0[3];
    for (int i = 0; i < 3; ++i) {
        const float u = (x[i] - g.mn[i]) * g.scale[i];
        const float fl = fminf(fmaxf(floorf(u), 0.0f), static_cast<float>(g.n[i] - 2));
        i0[i] = static_cast<int>(fl);
        f[i] = fminf(fmaxf(u - fl, 0.0f), 1.0f);
    }
    return (static_cast<int64_t>(i0[0]) * g.n[1] + i0[1]) * g.n[2] + i0[2];
}

__device__ __forceinline__ int64_t corner(const Tri& t, int c) {
    return t.base + ((c >> 2) & 1) * static_cast<int64_t>(t.sx) + ((c >> 1) & 1) * t.sy + (c & 1);
}

__device__ __forceinline__ float softplus_f(float x) {
    return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x)));
}
__device__ __forceinline__ float sigmoid_f(float x) { return 1.0f / (1.0f + expf(-x)); }

__device__ __forceinline__ int64_t live_count(const int64_t* n_kept, int64_t cap) {
    const int64_t n = *n_kept;
    return n < cap ? n : cap;
}

// ---------------------------------------------------------------------------
// prep: per-ray encodings and first-layer per-ray part
// ---------------------------------------------------------------------------
// base[r][i] = b1[i] + sum_q W1[i][view_col+q] * PE(d_r)[q];  pe[r] = [PE(d_r) (27), 1, 0, 0, 0, 0]
// (view_col: the view part's first column, after the per-sample inputs;
// w1_in: the row stride of W1)
// Per-call preparation, one workgroup role per block: the first
// kPackThreads/256 workgroups pack the network's operands; each following
// workgroup takes kPrepRays rays: 12 threads per ray evaluate its 24 sines
// and cosines once into LDS, then each thread forms one output of the first
// layer's view part for half of the rays; the last zblocks workgroups clear
// the backward's cell counts.
constexpr int kPrepRays = 16;   // rays per workgroup of the preparation
struct PrepArgs {
    PackArgs pk;
    const float* rays_d;
    int B;
    const float* w1;
    const float* b1;
    int w1_in;      // row stride of W1
    int view_col;   // first column of W1's view part
    float* base;
    float* pe;
    int* wide;      // MlpArgs::wide, cleared (NULL: none)
    float4* pad;    // the zero record, cleared (NULL: none)
    int* zero;      // cleared (NULL: none)
    int64_t nzero;
    int zblocks;
    int blocks;     // workgroups of the preparation
};

__device__ __forceinline__ void prep_body(const PrepArgs& P, int blk) {
    constexpr int kPackBlocks = kPackThreads / 256;
    if (blk < kPackBlocks) {
        if (blk == 0 && threadIdx.x == 0 && P.wide) *P.wide = 0;
        if (blk == 0 && threadIdx.x < 4 && P.pad) P.pad[threadIdx.x] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        pack_weights(P.pk, blk * 256 + threadIdx.x);
        return;
    }
    const int B = P.B, w1_in = P.w1_in, view_col = P.view_col, zblocks = P.zblocks;
    const float* __restrict__ rays_d = P.rays_d;
    const float* __restrict__ w1 = P.w1;
    const float* __restrict__ b1 = P.b1;
    float* __restrict__ base = P.base;
    float* __restrict__ pe = P.pe;
    int* __restrict__ zero = P.zero;
    const int64_t nzero = P.nzero;
    const int ray_blocks = (B + kPrepRays - 1) / kPrepRays;
    const int zb = blk - kPackBlocks - ray_blocks;
    if (zb >= 0) {   // the last zblocks workgroups clear `zero` (the backward's cell counts)
        const int64_t stride = static_cast<int64_t>(zblocks) * 256, first = static_cast<int64_t>(zb) * 256 + threadIdx.x;
        int64_t done = 0;
        if ((reinterpret_cast<uintptr_t>(zero) & 15u) == 0) {   // 16-byte stores, then the tail
            int4* z4 = reinterpret_cast<int4*>(zero);
            const int64_t n4 = nzero / 4;
            for (int64_t i = first; i < n4; i += stride) z4[i] = make_int4(0, 0, 0, 0);
            done = 4 * n4;
        }
        for (int64_t i = done + first; i < nzero; i += stride) zero[i] = 0;
        return;
    }
    __shared__ float se[kPrepRays][32];
    const int t = threadIdx.x;
    const int r0 = kPrepRays * (blk - kPackBlocks);
    if (t < 12 * kPrepRays) {
        const int rr = t / 12, q = t % 12, fq = q / 3, c = q % 3;
        const int r = r0 + rr;
        if (r < B) {
            const float dc = rays_d[3 * r + c];
            float sv, cv;
            sincosf(dc * static_cast<float>(1 << fq), &sv, &cv);
            se[rr][3 + 6 * fq + c] = sv;
            se[rr][6 + 6 * fq + c] = cv;
            if (fq == 0) se[rr][c] = dc;
        }
    }
    if (t < 5 * kPrepRays)   // entry 27: the first layer's constant input; 28..31 zero
        se[t / 5][kPE + t % 5] = t % 5 == 0 ? 1.0f : 0.0f;
    __syncthreads();
    // thread (h, i) forms output i for rays h, h + 2, ...; its weights stay in
    // registers across the rays
    const int h = t >> 7, i = t & (kH - 1);
    float wv[kPE];
    const float bi = w1 ? b1[i] : 0.0f;
    if (w1) {
        #pragma unroll
        for (int q = 0; q < kPE; ++q) wv[q] = w1[i * w1_in + view_col + q];
    }
    bool dead = w1 && !P.pk.bf16 && bi == 0.0f;   // (see kDeadBias)
    for (int q = 0; dead && q < w1_in; ++q) dead = w1[i * w1_in + q] == 0.0f;
    for (int rr = h; rr < kPrepRays; rr += 2) {
        const int r = r0 + rr;
        if (r >= B) break;
        if (w1) {
            float acc = bi;
            #pragma unroll
            for (int q = 0; q < kPE; ++q) acc += wv[q] * se[rr][q];
            if (dead) acc = kDeadBias;
            base[static_cast<int64_t>(r) * kH + i] = acc;
        }
        if (i < 32) pe[static_cast<int64_t>(r) * 32 + i] = se[rr][i];
    }
}

__global__ __launch_bounds__(256) void prep_kernel(PrepArgs P) { prep_body(P, blockIdx.x); }

// ---------------------------------------------------------------------------
// gather: raw density and interpolated features per sample
// ---------------------------------------------------------------------------
// A wavefront's LDS accesses are in order; the compiler is kept from moving them.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int kPerm>
__device__ __forceinline__ int quad_bcast(int x) {
    return __builtin_amdgcn_update_dpp(0, x, kPerm, 0xf, 0xf, true);
}

struct GatherArgs {
    SampleArgs sa;
    GridArgs g;
    const float* density;
    const void* feat;
    const int64_t* n_kept;
    int64_t cap;
    float* raw_out;
    float* feat_out;
};

// kFeat: 0 density only, 1 float32 features, 2 bfloat16 features.
// A wavefront takes 64 samples, each lane the cell of one, then 16 at a time,
// a lane quad each: lane e < 3 of the quad reads words e of the 8 corners'
// features, 4 values each, so that a quad's load covers a corner's features
// contiguously, and lane c the densities of corners 2c and 2c + 1 (neighbours
// along z).  With a sample per lane it was bound by the address unit: 24
// feature loads and 8 density loads of 64 separate addresses, where the quads
// need 8 of 16 segments and one.  387k training samples (160^3 cells, float32)
// 43 -> 34 us, 30653 rays of a preview image 134 -> 109; in bfloat16 it
// is bound by memory: 7.1M samples in 256^3 cells 452 -> 417 us (1.2 GB read,
// 0.45 written, 3.9 TB/s), 65536 rays of an image 137 -> 134.  Both z neighbours in
// one load (half the loads again) and a contiguous eighth of the samples per
// XCD were no faster (429, 128; 416, 133).  The sums keep their order.
template <int kFeat>
__device__ __forceinline__ void gather_body(const GatherArgs& a, int blk, int nblk) {
    struct Cell {
        float f[3];
        int pad;
        int64_t base;
    };
    __shared__ Cell cells[4][64];
    const int64_t n = live_count(a.n_kept, a.cap);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quad = lane >> 2, part = lane & 3;
    const int64_t sy = a.g.n[2], sx = static_cast<int64_t>(a.g.n[1]) * a.g.n[2];
    typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
    for (int64_t s0 = (static_cast<int64_t>(blk) * 4 + wave) * 64; s0 < n; s0 += static_cast<int64_t>(nblk) * 256) {
        {
            const int64_t s = s0 + lane < n ? s0 + lane : n - 1;
            float x[3];
            sample_point(a.sa, a.sa.sample_ray[s], a.sa.sample_k[s], x, nullptr);
            Cell c;
            c.base = cell_base(a.g, x, c.f);
            wave_lds_fence();   // the cells' last readers are done
            cells[wave][lane] = c;
            wave_lds_fence();
        }
        constexpr int kStep = 2;   // sample groups whose loads are in flight together
        #pragma unroll
        for (int u0 = 0; u0 < 4; u0 += kStep) {
            if (s0 + 16 * u0 >= n) break;
            f2u d[kStep];
            float4 q4[kFeat == 1 ? kStep : 1][8];
            uint2 q2[kFeat == 2 ? kStep : 1][8];
            float w[kStep][8];
            #pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const Cell c = cells[wave][16 * (u0 + u) + quad];
                const float gx[2] = {1.0f - c.f[0], c.f[0]}, gy[2] = {1.0f - c.f[1], c.f[1]},
                            gz[2] = {1.0f - c.f[2], c.f[2]};
                #pragma unroll
                for (int k = 0; k < 8; ++k) w[u][k] = gx[(k >> 2) & 1] * gy[(k >> 1) & 1] * gz[k & 1];
                d[u] = *reinterpret_cast<const f2u*>(a.density + c.base + (part & 2 ? sx : 0) + (part & 1 ? sy : 0));
                if (kFeat == 0 || part == 3) continue;
                #pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int64_t v = c.base + ((k >> 2) & 1) * sx + ((k >> 1) & 1) * sy + (k & 1);
                    if (kFeat == 1) q4[u][k] = (static_cast<const float4*>(a.feat) + part)[3 * v];
                    else q2[u][k] = (static_cast<const uint2*>(a.feat) + part)[3 * v];
                }
            }
            #pragma unroll
            for (int u = 0; u < kStep; ++u) {
                const int64_t s = s0 + 16 * (u0 + u) + quad;
                // corner 2c + z is in lane c's component z
                const int d0 = __float_as_int(d[u].x), d1 = __float_as_int(d[u].y);
                float raw = 0.0f;
                raw += w[u][0] * __int_as_float(quad_bcast<0x00>(d0));
                raw += w[u][1] * __int_as_float(quad_bcast<0x00>(d1));
                raw += w[u][2] * __int_as_float(quad_bcast<0x55>(d0));
                raw += w[u][3] * __int_as_float(quad_bcast<0x55>(d1));
                raw += w[u][4] * __int_as_float(quad_bcast<0xaa>(d0));
                raw += w[u][5] * __int_as_float(quad_bcast<0xaa>(d1));
                raw += w[u][6] * __int_as_float(quad_bcast<0xff>(d0));
                raw += w[u][7] * __int_as_float(quad_bcast<0xff>(d1));
                if (s >= n) continue;
                if (part == 3) a.raw_out[s] = raw;
                if (kFeat == 0 || part == 3) continue;
                float4 f = make_float4(0, 0, 0, 0);
                #pragma unroll
                for (int k = 0; k < 8; ++k) {
                    float4 v;
                    if (kFeat == 1) {
                        v = q4[u][k];
                    } else {
                        const uint2 b = q2[u][k];
                        v = make_float4(__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xFFFF0000u),
                                        __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xFFFF0000u));
                    }
                    f.x += w[u][k] * v.x;
                    f.y += w[u][k] * v.y;
                    f.z += w[u][k] * v.z;
                    f.w += w[u][k] * v.w;
                }
                reinterpret_cast<float4*>(a.feat_out + s * kC)[part] = f;
            }
        }
    }
}

__global__ __launch_bounds__(256) void density_gather_kernel(GatherArgs a) { gather_body<0>(a, blockIdx.x, gridDim.x); }

// The gather and the per-call preparation in one launch (the two are
// independent: the preparation's workgroups fill the gather's latency-bound
// schedule, 6-9 us per training step at the full configuration): the first
// gather_blocks workgroups gather, the others prepare.
template <int kFeat>
__global__ __launch_bounds__(256) void prep_gather_kernel(PrepArgs P, GatherArgs a, int gather_blocks) {
    const int blk = static_cast<int>(blockIdx.x);
    if (blk < gather_blocks) gather_body<kFeat>(a, blk, gather_blocks);
    else prep_body(P, blk - gather_blocks);
}

// ---------------------------------------------------------------------------
// compose: one wavefront per ray slot, 64 samples per step, prefix scans
// ---------------------------------------------------------------------------
struct ComposeArgs {
    SampleArgs sa;
    const int* perm;
    const int* ray_offset;
    const int* n_uniform;
    const int64_t* n_kept;
    int64_t cap;
    int B;
    float act_shift;
    float bg[3];
    float* raw;        // in: raw density; out (backward): dL/draw
    float* col;        // in: colour [cap][4]; out (backward): dL/dc
    int with_color;
    // forward outputs
    float* rgb;
    float* depth;
    float* acc;
    float* log_t_end;
    float* seg_w;
    float* sample_w;
    // forward, inside dvgo_train_step: the photometric loss's gradient and
    // each ray's loss (summed later in a fixed order); with w_pt or w_bg also
    // the per-point rgb and background entropy terms (the backward reads
    // target for the per-point term)
    const float* target;
    float* grad_rgb_out;
    float* sq_err;
    float w_pt, w_bg;
    // backward inputs
    const float* log_t_end_in;
    const float* grad_rgb;
    const float* grad_depth;
    const float* grad_acc;
    // backward binning by fine cell (cell_count == nullptr: off)
    GridArgs g;
    int* cell_count;       // [ncell + 1], zero on entry
    int2* cell_rank;       // [cap] (cell, rank within cell)
    float4* rec_head;      // [cap] (fx, fy, fz, dL/draw)
    // backward, float32 network: set where a |dL/dc| is 2^64 or more (NULL: off)
    int* wide;
    // forward without a network: each sample's raw density interpolated
    // here from this grid (on g) instead of read from raw
    const float* density_in;
};

// Fine cell of a point (its vertex (0,0,0)) and the fractional position f
// inside it, clamped like the trilinear interpolation.
__device__ __forceinline__ int cell_of(const GridArgs& g, const float x[3], float f[3]) {
    int i0[3];
    for (int i = 0; i < 3; ++i) {
        const float u = (x[i] - g.mn[i]) * g.scale[i];
        const float fl = fminf(fmaxf(floorf(u), 0.0f), static_cast<float>(g.n[i] - 2));
        i0[i] = static_cast<int>(fl);
        f[i] = fminf(fmaxf(u - fl, 0.0f), 1.0f);
    }
    return (i0[0] * (g.n[1] - 1) + i0[1]) * (g.n[2] - 1) + i0[2];
}

// What the fused adjoint takes over from the forward of its ray: per sample of
// the first kKeptSteps 64-sample steps w_k and the inclusive sum of
// sigma*delta in its step (each lane reads what it wrote), log T at the start
// of step j in lane j (steps below 64), dL/dC and log T_end.  4 KB per
// wavefront, so that 32 of them share a compute unit.
constexpr int kKeptSteps = 8;
struct KeptRay {
    float2* kept;   // [kKeptSteps][64]
    float start, g[3], log_t_end;
};

// Forward compositing of ray slot `slot` by one wavefront (segs: its 32
// segment sums in LDS).  With a.target it also forms the photometric
// gradient dL/dC; every lane returns that gradient and log T_end in K.
template <bool kInline, bool kKeep>   // kInline: the raw densities interpolated here (a.density_in)
__device__ __forceinline__ void compose_fwd_ray(const ComposeArgs& a, int slot, int lane, float* segs, KeptRay& K) {
    const int64_t n = live_count(a.n_kept, a.cap);
    const int r = a.perm[slot];
    int64_t s0 = a.ray_offset[slot], s1 = a.ray_offset[slot + 1];
    s0 = s0 < n ? s0 : n;
    s1 = s1 < n ? s1 : n;
    const int nu = a.n_uniform[r];
    const float tn = a.sa.t_near[r];
    const float p = a.sa.jitter ? a.sa.jitter[r] : 0.0f;
    const float step = a.sa.step;
    float ro[3] = {0.0f, 0.0f, 0.0f}, rd[3] = {0.0f, 0.0f, 0.0f};   // the ray, for the inline density
    if (kInline)
        for (int i = 0; i < 3; ++i) {
            ro[i] = a.sa.rays_o[3 * r + i];
            rd[i] = a.sa.rays_d[3 * r + i];
        }
    if (lane < 32) segs[lane] = 0.0f;
    __builtin_amdgcn_wave_barrier();
    float logT = 0.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f, dep = 0.0f, accw = 0.0f, ptl = 0.0f;
    float tg[3] = {0.0f, 0.0f, 0.0f};
    if (a.w_pt > 0.0f)
        for (int c = 0; c < 3; ++c) tg[c] = a.target[3 * r + c];
    for (int64_t base = s0; base < s1; base += 64) {
        const int64_t s = base + lane;
        const bool ok = s < s1;
        float sd = 0.0f, alpha = 0.0f, tk = 0.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
        int k = 0;
        if (ok) {
            k = a.sa.sample_k[s];
            tk = recipe_tk(tn, p, k, step);
            float raw;
            if (kInline) {   // the gather's interpolation, in its order
                float x[3];
                recipe_x(ro, rd, tk, x);
                const Tri t = trilinear(a.g, x);
                float dv[8];
                #pragma unroll
                for (int c = 0; c < 8; ++c) dv[c] = a.density_in[corner(t, c)];
                raw = 0.0f;
                #pragma unroll
                for (int c = 0; c < 8; ++c) raw += t.w[c] * dv[c];
            } else {
                raw = a.raw[s];
            }
            const float sig = softplus_f(raw + a.act_shift);
            sd = sig * step;
            alpha = -expm1f(-sd);
            if (a.with_color) {
                const float4 c = reinterpret_cast<const float4*>(a.col)[s];
                c0 = c.x; c1 = c.y; c2 = c.z;
            }
        }
        const float incl = wave_incl_scan(sd, lane);
        const float excl = dpp_wave<0x138>(incl);   // wave_shr:1, lane 0 reads 0
        const float w = ok ? expf(logT - excl) * alpha : 0.0f;
        if constexpr (kKeep) {
            const int64_t it = (base - s0) >> 6;
            if (lane == it) K.start = logT;
            if (it < kKeptSteps) K.kept[it * 64 + lane] = make_float2(w, incl);
        }
        cr += w * c0; cg += w * c1; cb += w * c2;
        dep += w * tk;
        accw += w;
        if (a.w_pt > 0.0f) {   // per-point rgb: w_k ||c_k - C*||^2
            const float e0 = c0 - tg[0], e1 = c1 - tg[1], e2 = c2 - tg[2];
            ptl += w * (e0 * e0 + e1 * e1 + e2 * e2);
        }
        if (ok && a.seg_w) atomicAdd(&segs[(32LL * k) / nu], w);
        if (ok && a.sample_w) a.sample_w[s] = w;
        logT -= lane_value(incl, 63);
    }
    cr = wave_sum(cr); cg = wave_sum(cg); cb = wave_sum(cb);
    dep = wave_sum(dep);
    accw = wave_sum(accw);
    if (a.w_pt > 0.0f) ptl = wave_sum(ptl);
    __builtin_amdgcn_wave_barrier();
    // the ray's colour and loss terms, in every lane (the stores from lane 0)
    const float T = expf(logT);
    K.g[0] = K.g[1] = K.g[2] = 0.0f;
    K.log_t_end = logT;
    if (a.rgb) {
        const float c3[3] = {cr + T * a.bg[0], cg + T * a.bg[1], cb + T * a.bg[2]};
        if (lane == 0) {
            a.rgb[3 * r + 0] = c3[0];
            a.rgb[3 * r + 1] = c3[1];
            a.rgb[3 * r + 2] = c3[2];
        }
        if (a.target) {   // Eq. photo_loss: gradient 2 (C - C*)/B, as dvgo_photo_loss forms it
            const float invB = 1.0f / static_cast<float>(a.B);
            float e2 = 0.0f;
            for (int c = 0; c < 3; ++c) {
                const float d = c3[c] - a.target[3 * r + c];
                K.g[c] = 2.0f * d * invB;
                e2 += d * d;
            }
            if (a.w_pt > 0.0f) e2 += a.w_pt * ptl;
            if (a.w_bg > 0.0f) {   // background entropy of T_end, clamped to [1e-6, 1 - 1e-6]
                const float pb = fminf(fmaxf(T, 1e-6f), 1.0f - 1e-6f);
                e2 += a.w_bg * (-pb * logf(pb) - (1.0f - pb) * log1pf(-pb));
            }
            if (lane == 0) {
                for (int c = 0; c < 3; ++c) a.grad_rgb_out[3 * r + c] = K.g[c];
                a.sq_err[r] = e2;
            }
        }
    }
    if (lane == 0) {
        if (a.depth) a.depth[r] = dep;
        if (a.acc) a.acc[r] = accw;
        a.log_t_end[r] = logT;
    }
    if (a.seg_w && lane < 32) a.seg_w[static_cast<int64_t>(r) * 32 + lane] = segs[lane];
}

// Wavefronts (rays) per workgroup of the compositing kernels: one, so that a
// long ray holds only its own slot (with four, a workgroup's resources stayed
// held until its longest ray was done: the training step's compositing took
// 1 us longer).
constexpr int kComposeWaves = 1;
constexpr int kComposeThreads = 64 * kComposeWaves;
inline dim3 compose_grid(int B) { return dim3((B + kComposeWaves - 1) / kComposeWaves); }

template <bool kInline>
__global__ __launch_bounds__(kComposeThreads) void compose_fwd_kernel(ComposeArgs a) {
    __shared__ float segs[kComposeWaves][32];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int slot = blockIdx.x * kComposeWaves + wave;
    if (slot >= a.B) return;
    KeptRay K;
    compose_fwd_ray<kInline, false>(a, slot, lane, segs[wave], K);
}

// Backward of compose: walk each ray from its end in 64-sample steps,
// carrying the suffix sums S.  The transmittance is recomputed from the
// samples' densities as the forward forms it, by prefix sums from the ray's
// start: log T at the start of each 64-sample step comes from a first pass
// over the ray's steps (lane j keeps the start of step j), so T_k, T_{k+1}
// and w_k are the forward's values bit for bit.  (Forming log T_k as
// log T_end plus the suffix of sigma*delta would cancel: with an optical
// depth D along the ray it loses D*2^-24 of absolute accuracy in log T.)
// Rays of more than 64 steps take the first pass once per group of 64.
__device__ __forceinline__ float sd_of(const ComposeArgs& a, int64_t s, int64_t s1) {
    return s < s1 ? softplus_f(a.raw[s] + a.act_shift) * a.sa.step : 0.0f;
}

// The adjoint of ray slot `slot` by one wavefront.  kFused: with what the
// forward has kept in K (no depth or opacity gradient then), else from
// a.grad_* and a.log_t_end_in.
template <bool kFused>
__device__ __forceinline__ void compose_bwd_ray(const ComposeArgs& a, int slot, int lane, const KeptRay& K) {
    constexpr int kCh = kFused ? 3 : 5;   // channels: colour; depth and opacity
    const int64_t n = live_count(a.n_kept, a.cap);
    const int r = a.perm[slot];
    int64_t s0 = a.ray_offset[slot], s1 = a.ray_offset[slot + 1];
    s0 = s0 < n ? s0 : n;
    s1 = s1 < n ? s1 : n;
    // (r < 0 never holds; testing it keeps the ray's load in flight with
    // the offsets' instead of after this test)
    if (s1 <= s0 || r < 0) return;
    const float tn = a.sa.t_near[r];
    const float p = a.sa.jitter ? a.sa.jitter[r] : 0.0f;
    const float step = a.sa.step;
    float g[5];
    for (int c = 0; c < 3; ++c) g[c] = kFused ? K.g[c] : a.grad_rgb ? a.grad_rgb[3 * r + c] : 0.0f;
    g[3] = !kFused && a.grad_depth ? a.grad_depth[r] : 0.0f;
    g[4] = !kFused && a.grad_acc ? a.grad_acc[r] : 0.0f;
    float ro[3] = {0.0f, 0.0f, 0.0f}, rd[3] = {0.0f, 0.0f, 0.0f};   // the ray, for the binning
    if (a.cell_count) {
        for (int i = 0; i < 3; ++i) {
            ro[i] = a.sa.rays_o[3 * r + i];
            rd[i] = a.sa.rays_d[3 * r + i];
        }
    }
    const float Tend = expf(kFused ? K.log_t_end : a.log_t_end_in[r]);
    bool wide = false;   // this lane has seen a |dL/dc| out of the planes' range
    float S[5] = {Tend * a.bg[0], Tend * a.bg[1], Tend * a.bg[2], 0.0f, 0.0f};
    // auxiliary losses: the background entropy's gradient on T_end reaches
    // every sample through dT_end/dsigma_k = -delta T_end; the per-point rgb
    // loss adds 2 w_pt w_k (c_k - C*)/B to each colour's gradient
    const float invB = 1.0f / static_cast<float>(a.B);
    float dsig_bg = 0.0f;
    if (a.w_bg > 0.0f && Tend > 1e-6f && Tend < 1.0f - 1e-6f)
        dsig_bg = -Tend * a.w_bg * (log1pf(-Tend) - logf(Tend)) * invB;
    float tg[3] = {0.0f, 0.0f, 0.0f};
    if (a.w_pt > 0.0f)
        for (int c = 0; c < 3; ++c) tg[c] = a.target[3 * r + c];
    const float ptk = 2.0f * a.w_pt * invB;
    const int64_t nsteps = (s1 - s0 + 63) / 64;
    const int64_t ngroups = (nsteps + 63) / 64;
    for (int64_t grp = ngroups - 1; grp >= 0; --grp) {
        // log T at the start of steps 64*grp .. 64*grp+63, lane j holding step 64*grp+j
        const int64_t first = 64 * grp, last = first + 63 < nsteps - 1 ? first + 63 : nsteps - 1;
        float start = 0.0f;
        if (kFused && grp == 0) {
            start = K.start;
        } else {
            float logT = 0.0f;
            for (int64_t j = 0; j < last; ++j) {
                if (j >= first && lane == static_cast<int>(j - first)) start = logT;
                logT -= wave_sum(sd_of(a, s0 + j * 64 + lane, s1));
            }
            if (lane == static_cast<int>(last - first)) start = logT;
        }
        for (int64_t it = last; it >= first; --it) {
            const int64_t s = s0 + it * 64 + lane;
            const bool ok = s < s1;
            float sd = 0.0f, raw = 0.0f, tk = 0.0f, v[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            if (ok) {
                raw = a.raw[s];
                tk = recipe_tk(tn, p, a.sa.sample_k[s], step);
                if (a.with_color) {
                    const float4 c = reinterpret_cast<const float4*>(a.col)[s];
                    v[0] = c.x; v[1] = c.y; v[2] = c.z;
                }
                v[3] = tk;
                v[4] = 1.0f;
            }
            const float logT0 = lane_value(start, static_cast<int>(it - first));
            float incl, w;
            if (kFused && it < kKeptSteps) {
                const float2 kept = K.kept[it * 64 + lane];
                w = kept.x;
                incl = kept.y;
            } else {
                if (ok) sd = softplus_f(raw + a.act_shift) * step;
                incl = wave_incl_scan(sd, lane);
                const float excl = dpp_wave<0x138>(incl);   // wave_shr:1, lane 0 reads 0
                w = ok ? expf(logT0 - excl) * -expm1f(-sd) : 0.0f;   // T_k alpha_k, as the forward
            }
            const float Tafter = expf(logT0 - incl);     // T_{k+1}
            float dsig = dsig_bg;
            float tot[5];
            for (int ch = 0; ch < kCh; ++ch) {
                const float wv = w * v[ch];
                const float sfx = wave_incl_suffix(wv, lane);
                const float sfx_ex = dpp_wave<0x130>(sfx);   // wave_shl:1, lane 63 reads 0
                dsig += g[ch] * (Tafter * v[ch] - (S[ch] + sfx_ex));
                tot[ch] = lane_value(sfx, 0);
            }
            const float draw = step * dsig * sigmoid_f(raw + a.act_shift);
            if (ok) {
                a.raw[s] = draw;
                if (a.with_color) {
                    float4 dc = make_float4(w * g[0], w * g[1], w * g[2], 0.0f);
                    if (a.w_pt > 0.0f) {
                        dc.x += ptk * w * (v[0] - tg[0]);
                        dc.y += ptk * w * (v[1] - tg[1]);
                        dc.z += ptk * w * (v[2] - tg[2]);
                    }
                    reinterpret_cast<float4*>(a.col)[s] = dc;
                    wide |= !(fabsf(dc.x) + fabsf(dc.y) + fabsf(dc.z) < 0x1p64f);
                }
            }
            if (a.cell_count) {   // bin the sample by fine cell (wave-uniform branch)
                int cell = -1;
                if (ok) {
                    float x[3], f[3];
                    recipe_x(ro, rd, tk, x);   // the sample's point, as sample_point forms it
                    cell = cell_of(a.g, x, f);
                    a.rec_head[s] = make_float4(f[0], f[1], f[2], draw);
                }
                const int rank = run_rank(cell, ok, lane, a.cell_count);
                if (ok) a.cell_rank[s] = make_int2(cell, rank);
            }
            for (int ch = 0; ch < kCh; ++ch) S[ch] += tot[ch];
        }
    }
    if (a.wide && __any(wide) && lane == 0) *a.wide = 1;
}

__global__ __launch_bounds__(kComposeThreads) void compose_bwd_kernel(ComposeArgs a) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int slot = blockIdx.x * kComposeWaves + wave;
    if (slot >= a.B) return;
    compose_bwd_ray<false>(a, slot, lane, KeptRay{});
}

// The training step's compositing and its adjoint in one launch: each
// wavefront composites its ray (forward outputs, loss terms, dL/dC), then
// walks it back with what it has kept.  The adjoint of a ray depends only on
// that ray's forward, so no other wavefront waits.  Bound by vector
// instructions (71 % of the issue slots): forming T_k and w_k again, and log T
// at the steps' starts by a pass of their own, were a third of them.  7.1M
// samples 269 -> 238 us, 387k 34 -> 26, 106k 13.8 -> 11.6.
__global__ __launch_bounds__(kComposeThreads) void compose_step_kernel(ComposeArgs fa, ComposeArgs ba) {
    __shared__ float segs[kComposeWaves][32];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int slot = blockIdx.x * kComposeWaves + wave;
    if (slot >= fa.B) return;
    __shared__ float2 kept[kComposeWaves][kKeptSteps * 64];
    KeptRay K;
    K.kept = kept[wave];
    K.start = 0.0f;
    compose_fwd_ray<false, true>(fa, slot, lane, segs[wave], K);
    compose_bwd_ray<true>(ba, slot, lane, K);
}

// ---------------------------------------------------------------------------
// scatter: transpose of the trilinear gathers, without float atomics.
// Samples are counting-sorted by fine cell (one integer atomic per run of
// equal cells in a wavefront), then one lane quad per grid vertex sums the
// contributions of the samples in its 8 neighbouring cells and adds them to
// the gradient with a plain read-modify-write.
// ---------------------------------------------------------------------------
struct BinArgs {
    SampleArgs sa;
    GridArgs g;
    const int64_t* n_kept;
    int64_t cap;
    int* cell_count;       // [ncell + 1]
    const int* cell_start; // [ncell + 1]
    int2* cell_rank;       // [cap] (cell, rank within cell)
    const float4* rec_head;  // [cap] (fx, fy, fz, draw)
    int with_feat;         // records carry dL/dfeat
    float4* rec;           // [cap][4] in binned order: (fx, fy, fz, draw), df[0..11]
    float* grad_density;
    float* grad_feat;
    int64_t ncell;
};

// Records in binned order when no network backward places them (density
// only): the head (fractional position, dL/draw) at cell start + rank.  The
// zero record as well, which the network's preparation clears otherwise.
__global__ __launch_bounds__(256) void bin_place_kernel(BinArgs a) {
    if (blockIdx.x == 0 && threadIdx.x < 4) a.rec[4 * a.cap + threadIdx.x] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const int64_t n = live_count(a.n_kept, a.cap);
    for (int64_t s = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; s < n;
         s += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int2 cr = a.cell_rank[s];
        const int64_t pos = static_cast<int64_t>(a.cell_start[cr.x]) + cr.y;
        a.rec[pos * 4] = a.rec_head[s];
    }
}

// Gradients of a wavefront's 16 consecutive vertices, a lane quad each.  Vertex
// (i,j,k) is corner (dx,dy,dz) of cell (i-dx, j-dy, k-dz); the samples binned
// in those cells are summed with the vertex's trilinear weight.  For each
// (dx,dy) the cells k-1 (dz = 1) and k (dz = 0) are neighbours in the cell
// order, so their records form one run, split at the start of cell k: lane
// 2dx + dy of the quad finds it and lists its records in LDS.  Then the quad
// reads each record as one 64-byte segment (lane `part` its word `part`: the
// density's, or four features'), kPairsAhead of them in flight.
//
// With a vertex per lane, a step of the longest run cost four load
// instructions with 9 of 64 lanes active: the address units, busy 72 % of the
// time, bounded the walk.  With the Adam step: 106k samples in 31^3 cells
// 34 -> 17 us, 153k in 99^3 65 -> 57, 387k in 159^3 183 -> 175, 7.1M in 255^3
// 1600 -> 1494 (1460 in the shares of grid_adam_blocks; 5.7 GB of parameters
// and moments are 1040 us); the plain gather in 127^3 cells 70 -> 53.  Eight records ahead in fewer wavefronts:
// 14.5, 58, 191, 1520 us.  Four vertices per quad, their sums through LDS,
// take fewer loads (7.1M samples 1390 us) but a quarter of the wavefronts: 57
// us for the first of these.  Sums by LDS float atomics, in any split, were slower than
// either (64 lanes of one take as many cycles).
constexpr int kPairs = 32;       // records of a vertex listed at a time
constexpr int kPairsAhead = 4;

struct PairList {
    // x: record; y: 1 - (dx, dy, dz) in bytes 0..2
    uint2 pair[16][kPairs + 1];
};

struct VertexRun {
    int p0, pm, p1;   // this lane's run
};

// Whether any of the quad's lanes has a record.
__device__ __forceinline__ bool run_touched(const VertexRun& R) {
    const int any = R.p1 > R.p0;
    return (quad_bcast<0x00>(any) | quad_bcast<0x55>(any) | quad_bcast<0xaa>(any) | quad_bcast<0xff>(any)) != 0;
}

// Division of a vertex index by a grid extent, for wavefront-uniform operands
// (the host refuses grids of 2^31 vertices and more).
struct GridDivisor {
    uint32_t d, inv;
    __device__ explicit GridDivisor(int n) : d(n), inv(0xffffffffu / static_cast<uint32_t>(n)) {}
    __device__ uint32_t operator()(uint32_t x) const {
        uint32_t q = static_cast<uint32_t>(static_cast<uint64_t>(x) * inv >> 32);   // one or two too small
        q += x - q * d >= d;
        return q + (x - q * d >= d);
    }
};

// v0: the wavefront's first vertex (uniform); vertices beyond nv have no runs.
__device__ __forceinline__ VertexRun vertex_run(const BinArgs& a, GridDivisor by_nz, GridDivisor by_ny, uint32_t v0,
                                                int64_t nv) {
    const int lane = threadIdx.x & 63, c = lane & 3;
    const int nx = a.g.n[0], ny = a.g.n[1], nz = a.g.n[2], cy = ny - 1, cz = nz - 1;
    const uint32_t line = by_nz(v0);
    int i = static_cast<int>(by_ny(line)), j = static_cast<int>(line - i * static_cast<uint32_t>(ny));
    int k = static_cast<int>(v0 - line * static_cast<uint32_t>(nz)) + (lane >> 2);
    while (k >= nz) {   // at most 16 / nz times
        k -= nz;
        if (++j == ny) {
            j = 0;
            ++i;
        }
    }
    const int ci = i - (c >> 1), cj = j - (c & 1);
    VertexRun R;
    R.p0 = R.pm = R.p1 = 0;
    if (v0 + static_cast<int64_t>(lane >> 2) < nv && ci >= 0 && cj >= 0 && ci < nx - 1 && cj < cy) {
        const int row = (ci * cy + cj) * cz;
        R.p0 = a.cell_start[row + max(k - 1, 0)];   // cells k-1 and k, where they exist
        R.pm = a.cell_start[row + k];
        R.p1 = a.cell_start[row + min(k + 1, cz)];
    }
    return R;
}

// The whole wavefront calls this: word `part` of the quad's vertex's sums
// (part 0: density in .w).
__device__ __forceinline__ float4 vertex_sum(const BinArgs& a, VertexRun R, PairList& S) {
    const int lane = threadIdx.x & 63, part = lane & 3;
    uint2* list = S.pair[lane >> 2];
    const uint32_t y0 = (1u - (part >> 1)) | (1u - (part & 1)) << 8 | 1u << 16, y1 = y0 & 0xffffu;
    const float4* rec = a.rec + part;
    const uint32_t pad = static_cast<uint32_t>(a.cap);
    float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    bool more = R.p1 > R.p0;
    while (__any(more)) {
        // this lane's records, after those of the lanes before it
        const int n = min(R.p1 - R.p0, kPairs);
        const int n0 = quad_bcast<0x00>(n), n1 = quad_bcast<0x55>(n), n2 = quad_bcast<0xaa>(n),
                  n3 = quad_bcast<0xff>(n);
        const int at = (part > 0 ? n0 : 0) + (part > 1 ? n1 : 0) + (part > 2 ? n2 : 0);
        const int total = min(n0 + n1 + n2 + n3, kPairs);
        const int take = max(min(n, kPairs - at), 0);
        wave_lds_fence();   // the list's last readers are done
        for (int i = 0; i < take; ++i)
            list[at + i] = make_uint2(static_cast<uint32_t>(R.p0 + i), R.p0 + i < R.pm ? y1 : y0);
        R.p0 += take;
        more = R.p1 > R.p0;
        wave_lds_fence();
        // (no branch per record: the loads are to be in flight together)
        for (int b = 0; b < total; b += kPairsAhead) {
            uint32_t y[kPairsAhead];
            float4 r[kPairsAhead];
            const bool all = __any(b + kPairsAhead / 2 < total);
            #pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half && !all) break;
                #pragma unroll
                for (int u = half * kPairsAhead / 2; u < (half + 1) * kPairsAhead / 2; ++u) {
                    const uint2 x = list[min(b + u, total - 1)];
                    y[u] = x.y;
                    // beyond the list the zero record (a listed one times 0 is NaN where it is infinite)
                    r[u] = rec[static_cast<uint64_t>(b + u < total ? x.x : pad) * 4];
                }
            }
            #pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half && !all) break;
                #pragma unroll
                for (int u = half * kPairsAhead / 2; u < (half + 1) * kPairsAhead / 2; ++u) {
                    // dx ? fx : 1 - fx as |fx - (1 - dx)| (the position in the cell is in [0, 1])
                    const float w0 = fabsf(r[u].x - static_cast<float>(y[u] & 255u)) *
                                     fabsf(r[u].y - static_cast<float>(y[u] >> 8 & 255u)) *
                                     fabsf(r[u].z - static_cast<float>(y[u] >> 16 & 255u));
                    const float w = __int_as_float(quad_bcast<0x00>(__float_as_int(w0)));   // lane 0 holds the head
                    acc.x += w * r[u].x;
                    acc.y += w * r[u].y;
                    acc.z += w * r[u].z;
                    acc.w += w * r[u].w;
                }
            }
        }
    }
    return acc;
}

// Adds the vertices' gradients into the gradient grids.
__global__ __launch_bounds__(256) void vertex_gather_kernel(BinArgs a) {
    __shared__ PairList lists[4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = lane & 3;
    const int64_t nv = static_cast<int64_t>(a.g.n[0]) * a.g.n[1] * a.g.n[2];
    const GridDivisor by_nz(a.g.n[2]), by_ny(a.g.n[1]);
    for (int64_t v0 = static_cast<int64_t>(blockIdx.x) * 64 + 16 * wave; v0 < nv;
         v0 += static_cast<int64_t>(gridDim.x) * 64) {
        const VertexRun R = vertex_run(a, by_nz, by_ny, static_cast<uint32_t>(v0), nv);
        const bool touched = run_touched(R);
        if (!__any(touched)) continue;
        const float4 g = vertex_sum(a, R, lists[wave]);
        if (!touched) continue;
        const int64_t v = v0 + (lane >> 2);
        if (part == 0) {
            a.grad_density[v] += g.w;
        } else if (a.with_feat) {
            float4* gf = reinterpret_cast<float4*>(a.grad_feat + v * kC) + part - 1;
            float4 o = *gf;
            o.x += g.x;
            o.y += g.y;
            o.z += g.z;
            o.w += g.w;
            *gf = o;
        }
    }
}

// Grid parameters with their Adam moments, updated in place.
struct GridAdamArgs {
    float* pd;
    float* md;
    float* vd;
    float* pf;
    float* mf;
    float* vf;
    uint16_t* shadow;
    uint32_t* active;   // per-vertex bit: moments may be non-zero (NULL: every vertex steps)
    dvgo::AdamCoef c;
};

// Vertices of a chunk: what an XCD takes at a time (two x-planes).
__host__ __device__ inline int64_t adam_chunk(int ny, int nz) {
    return (2 * static_cast<int64_t>(ny) * nz + 255) / 256 * 256;
}

// The vertices' gradients as in vertex_gather_kernel, then the Adam step of
// their densities and features (and their bfloat16 copy), each lane on the
// values it has summed; a vertex no sample touches takes the step with a zero
// gradient, as dense Adam does.  The gradient never reaches memory.  A
// wavefront's 16 vertices own 768 consecutive bytes of each feature stream,
// six whole lines, which go past the caches; of a density stream they own half
// a line, which is left to the L2 to join with the neighbour's (past the caches
// as well, a grid that few samples touch took longer than with 64 vertices per
// wavefront: 128 rays in 255^3 cells 718 us against 595, now 667; 64 rays in
// 189^3 279, 260, 254; 512 rays in 147^3 145, 132, 133).
//
// With an activity mask, a vertex whose bit is clear (both moments zero)
// and that no sample touches is skipped: its step would compute m = v = 0
// and p - lr * 0 / (0 + eps) = p, so skipping it changes no bit, and its
// parameters and moments are neither read nor written.  A vertex that takes
// a step with any non-zero gradient gets its bit set.
__device__ __forceinline__ void vertex_adam_body(const BinArgs& a, const GridAdamArgs& o, int blk, int nblk) {
    __shared__ PairList lists[4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int vl = lane >> 2, part = lane & 3;
    const int ny = a.g.n[1], nz = a.g.n[2];
    const int64_t nv = static_cast<int64_t>(a.g.n[0]) * ny * nz;
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    f4* P = reinterpret_cast<f4*>(o.pf);
    f4* M = reinterpret_cast<f4*>(o.mf);
    f4* V = reinterpret_cast<f4*>(o.vf);
    u2* shadow = reinterpret_cast<u2*>(o.shadow);
    uint16_t* active = reinterpret_cast<uint16_t*>(o.active);   // a wavefront's 16 bits
    // Workgroups are dealt to the 8 XCDs round robin (block b on XCD b % 8).
    // The vertices are cut into chunks of two x-planes (rounded up to a
    // multiple of 256), dealt to the XCDs round robin as well: a cell's
    // records and start are read by the vertices of two neighbouring
    // x-planes, which then mostly sit in one chunk and so in one XCD's L2,
    // and every XCD gets an even share of the grid's busy middle (its
    // vertices with moments and samples) and of its idle rim.  The blocks of
    // an XCD walk its chunks in 64-vertex steps.  gridDim.x is a multiple of
    // 8; every wave's first vertex is a multiple of 16, so a wave owns a
    // half word of the activity mask.
    const int64_t kChunk = adam_chunk(ny, nz);
    const int xcd = blk & 7, nloc = nblk >> 3, loc = blk >> 3;
    const int64_t nchunk = (nv + kChunk - 1) / kChunk;
    const int64_t mine = nchunk > xcd ? (nchunk - xcd + 7) / 8 : 0;   // chunks of this XCD
    const GridDivisor by_nz(nz), by_ny(ny);
    int64_t chunk = 0, in_chunk = static_cast<int64_t>(loc) * 64;
    // the wave's first vertex of each step (nv: none left), increasing
    auto first_vertex = [&]() -> int64_t {
        while (in_chunk >= kChunk) {
            in_chunk -= kChunk;
            ++chunk;
        }
        const int64_t v0 = (chunk * 8 + xcd) * kChunk + in_chunk + 16 * wave;
        in_chunk += static_cast<int64_t>(nloc) * 64;
        return chunk < mine && v0 < nv ? v0 : nv;
    };
    // a step's runs and activity bits are loaded a step ahead
    VertexRun ahead;
    uint32_t bits_ahead = 0xffffu;
    auto load_ahead = [&](int64_t v0) {
        ahead.p0 = ahead.pm = ahead.p1 = 0;
        if (v0 >= nv) return;
        if (a.cell_start) ahead = vertex_run(a, by_nz, by_ny, static_cast<uint32_t>(v0), nv);   // else no samples
        if (active) bits_ahead = active[v0 >> 4];
    };
    int64_t next = first_vertex();
    load_ahead(next);
    while (next < nv) {
        const int64_t v0 = next;
        const int64_t v = v0 + vl;
        const VertexRun R = ahead;
        const uint32_t was = bits_ahead;
        const bool was_active = v < nv && ((was >> vl) & 1u);
        const bool touched = run_touched(R);
        const bool need = was_active || touched;
        next = first_vertex();
        load_ahead(next);
        if (!__any(need)) continue;
        // the parameters' streams, in flight while the records are summed
        f4 pq, mq, vq;
        if (need) {
            if (part) {
                const int64_t at = 3 * v + part - 1;
                pq = __builtin_nontemporal_load(P + at);
                mq = __builtin_nontemporal_load(M + at);
                vq = __builtin_nontemporal_load(V + at);
            } else {
                pq[3] = o.pd[v];
                mq[3] = o.md[v];
                vq[3] = o.vd[v];
            }
        }
        float4 g = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (__any(touched)) g = vertex_sum(a, R, lists[wave]);
        const float gg[4] = {g.x, g.y, g.z, g.w};
        if (need) {
            #pragma unroll
            for (int e = 0; e < 4; ++e) {
                float pe = pq[e], me = mq[e], ve = vq[e];
                dvgo::adam_update(o.c, pe, gg[e], me, ve);
                pq[e] = pe;
                mq[e] = me;
                vq[e] = ve;
            }
            if (part) {
                const int64_t at = 3 * v + part - 1;
                __builtin_nontemporal_store(pq, P + at);
                __builtin_nontemporal_store(mq, M + at);
                __builtin_nontemporal_store(vq, V + at);
                if (shadow) {
                    const uint2 b = dvgo::bf16x4_result(make_float4(pq.x, pq.y, pq.z, pq.w));
                    u2 bv;
                    bv.x = b.x;
                    bv.y = b.y;
                    __builtin_nontemporal_store(bv, shadow + at);
                }
            } else {
                o.pd[v] = pq[3];
                o.md[v] = mq[3];
                o.vd[v] = vq[3];
            }
        }
        if (active && __any(touched)) {   // (bits are only ever set)
            const int nonzero = touched && (g.w != 0.0f || (part && (g.x != 0.0f || g.y != 0.0f || g.z != 0.0f)));
            const uint64_t now = __ballot(quad_bcast<0x00>(nonzero) | quad_bcast<0x55>(nonzero) |
                                          quad_bcast<0xaa>(nonzero) | quad_bcast<0xff>(nonzero));
            uint32_t bits = 0;   // the quads' bits, gathered to one half word
            #pragma unroll
            for (int q = 0; q < 16; ++q) bits |= static_cast<uint32_t>(now >> (4 * q) & 1u) << q;
            if (bits & ~was && lane == 0) active[v0 >> 4] = static_cast<uint16_t>(was | bits);
        }
    }
}

__global__ __launch_bounds__(256, 6) void vertex_adam_kernel(BinArgs a, GridAdamArgs o) {
    vertex_adam_body(a, o, blockIdx.x, gridDim.x);
}

// Activity mask from given moments: bit v set iff any of vertex v's 26
// moments (density and 12 features, m and v) is non-zero.  Each wave covers
// 64 consecutive vertices, two whole words.
__global__ __launch_bounds__(256) void grid_active_kernel(const float* __restrict__ md, const float* __restrict__ vd,
                                                          const float* __restrict__ mf, const float* __restrict__ vf,
                                                          int64_t nv, uint32_t* __restrict__ active) {
    const int lane = threadIdx.x & 63;
    for (int64_t v0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + (threadIdx.x & ~63); v0 < nv;
         v0 += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t v = v0 + lane;
        bool nz = false;
        if (v < nv) {
            nz = md[v] != 0.0f || vd[v] != 0.0f;
            const float4* a = reinterpret_cast<const float4*>(mf + v * kC);
            const float4* b = reinterpret_cast<const float4*>(vf + v * kC);
            #pragma unroll
            for (int q = 0; q < 3; ++q) {
                const float4 x = a[q], y = b[q];
                nz |= x.x != 0.0f || x.y != 0.0f || x.z != 0.0f || x.w != 0.0f;
                nz |= y.x != 0.0f || y.y != 0.0f || y.z != 0.0f || y.w != 0.0f;
            }
        }
        const uint64_t bits = __ballot(nz);
        if (lane == 0) active[v0 >> 5] = static_cast<uint32_t>(bits);
        if (lane == 1 && v0 + 32 < nv) active[(v0 >> 5) + 1] = static_cast<uint32_t>(bits >> 32);
    }
}

// Deterministic sum of the per-block weight-gradient partials (+= into out):
// 64 parameters per workgroup, 16 wavefronts each summing every 16th
// partial row (all its loads issued before the sum, which keeps the row
// order), then a fixed-order sum of the 16 (deterministic).  With
// sq_err, workgroup 0 also forms the photometric loss (1/B) sum of the
// rays' squared errors, in a fixed order.
// With net.param, the summed gradient also takes the network's Adam step
// (the update dvgo_adam_step makes, on the same float32 gradient) and out
// is left zero.
struct NetAdam {
    float* param;
    float* m;
    float* v;
    dvgo::AdamCoef c;
};

struct ReduceArgs {
    const float* partial;   // [nblk][pstride]
    int nblk, nparams, pstride;
    float* out;             // the flat gradient (accumulated), or zeroed after the Adam step
    const float* sq_err;    // per-ray squared errors (NULL: no loss)
    int B;
    float* loss;
    NetAdam net;
};

// Workgroup blk (256 threads) sums the partials of parameters blk*64 ..
// blk*64 + 63 in a fixed order: wavefront w takes rows w, w + 4, ...
// (sixteen loads in flight at a time), then wavefront 0 adds the four sums
// in order; with net.param it then takes the Adam step.  Workgroup 0 also
// sums the squared errors into the loss.
__device__ __forceinline__ void reduce_body(const ReduceArgs& R, int blk) {
    __shared__ float sh[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = blk * 64 + lane;
    const int nblk = R.nblk, nparams = R.nparams, pstride = R.pstride, B = R.B;
    const float* __restrict__ partial = R.partial;
    float* __restrict__ out = R.out;
    const float* __restrict__ sq_err = R.sq_err;
    const NetAdam& net = R.net;
    static_assert(kMaxBwdBlocks <= 4 * 64, "a wavefront sums at most 64 partial rows");
    float s = 0.0f;
    if (p < nparams) {
        #pragma unroll
        for (int u0 = 0; u0 < 64; u0 += 16) {
            float v[16];
            #pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int b = wave + 4 * (u0 + u);
                v[u] = b < nblk ? partial[static_cast<int64_t>(b) * pstride + p] : 0.0f;
            }
            #pragma unroll
            for (int u = 0; u < 16; ++u) s += v[u];
        }
    }
    sh[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && p < nparams) {
        float t = 0.0f;
        for (int w = 0; w < 4; ++w) t += sh[w][lane];
        const float g = out[p] + t;
        if (net.param) {
            float pp = net.param[p], mm = net.m[p], vv = net.v[p];
            dvgo::adam_update(net.c, pp, g, mm, vv);
            net.param[p] = pp;
            net.m[p] = mm;
            net.v[p] = vv;
            out[p] = 0.0f;
        } else {
            out[p] = g;
        }
    }
    if (blk == 0 && sq_err) {
        __syncthreads();
        float e = 0.0f;
        for (int i0 = threadIdx.x; i0 < B; i0 += 256 * 8) {   // eight loads in flight, summed in order
            float v[8];
            #pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = i0 + 256 * u < B ? sq_err[i0 + 256 * u] : 0.0f;
            #pragma unroll
            for (int u = 0; u < 8; ++u) e += v[u];
        }
        for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
        if (lane == 0) sh[0][wave] = e;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.0f;
            for (int w = 0; w < 4; ++w) t += sh[0][w];
            if (R.loss) *R.loss = t * (1.0f / static_cast<float>(B));
        }
    }
}

__global__ __launch_bounds__(256) void reduce_partials_kernel(ReduceArgs R) { reduce_body(R, blockIdx.x); }

// The fused grid Adam and the reduction of the network's gradient partials
// in one launch (independent of each other): the first vblocks workgroups
// step the grids, the rest reduce, filling the grid step's tail.
__global__ __launch_bounds__(256, 6) void vertex_adam_reduce_kernel(BinArgs a, GridAdamArgs o, int vblocks,
                                                                 ReduceArgs R) {
    const int blk = static_cast<int>(blockIdx.x);
    if (blk < vblocks) vertex_adam_body(a, o, blk, vblocks);
    else reduce_body(R, blk - vblocks);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct Common {
    SampleArgs sa;
    GridArgs g;
    WsLayout L;
    char* ws;
    int64_t cap;
    int B;
    float box_min[3], box_max[3];
};

int32_t validate(const dvgo_field* field, const dvgo_mlp* mlp, const float* rays_o, const float* rays_d,
                 const float* t_near, const int32_t* n_uniform, const int32_t* perm, const int32_t* ray_offset,
                 const int32_t* sample_ray, const int32_t* sample_k, const int64_t* n_kept, int64_t capacity,
                 int32_t B, float step, const float* bg, void* workspace, size_t workspace_bytes,
                 bool forward_only = false) {
    if (!field || !bg || B < 0 || capacity < 0 || !(step > 0.0f)) return DVGO_E_ARG;
    if (!dvgo::box_ok(&field->box, 2) || !field->density) return DVGO_E_ARG;
    // vertex and cell indices, cell starts and record positions are int32
    if (static_cast<int64_t>(field->box.n[0]) * field->box.n[1] * field->box.n[2] >= (1LL << 31))
        return DVGO_E_UNSUPPORTED;
    if (mlp) {
        if (field->channels != kC) return DVGO_E_SHAPE;
        if (!field->feat) return DVGO_E_ARG;
        if (field->feat_dtype != DVGO_F32 && field->feat_dtype != DVGO_BF16) return DVGO_E_DTYPE;
        if (mlp->hidden != kH) return DVGO_E_SHAPE;
        if (mlp->precision != DVGO_F32 && mlp->precision != DVGO_BF16) return DVGO_E_DTYPE;
        if (mlp->pe_x != 0 && mlp->pe_x != kMaxKX) return DVGO_E_UNSUPPORTED;
        if (!mlp->w1 || !mlp->b1 || !mlp->w2 || !mlp->b2 || !mlp->w3 || !mlp->b3) return DVGO_E_ARG;
    }
    if (B > 0 && (!rays_o || !rays_d || !t_near || !n_uniform || !perm || !ray_offset)) return DVGO_E_ARG;
    if (!n_kept) return DVGO_E_ARG;
    if (capacity > 0 && (!sample_ray || !sample_k)) return DVGO_E_ARG;
    const size_t need = forward_only ? dvgo_render_fwd_workspace_bytes(B, capacity, kC, &field->box)
                        : mlp && mlp->precision == DVGO_F32
                            ? dvgo_render_workspace_bytes(B, capacity, kC, &field->box)
                            : dvgo_render_bf16_workspace_bytes(B, capacity, kC, &field->box);
    if (workspace_bytes < need || (!workspace && workspace_bytes)) return DVGO_E_CAPACITY;
    return DVGO_OK;
}

int grid_for(int64_t work, int per_block, int max_blocks) {
    int64_t b = (work + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return static_cast<int>(b);
}

// Host-side checks of a dvgo_grid_adam and its kernel arguments.
int32_t grid_adam_args(const dvgo_grid_adam* opt, GridAdamArgs* o) {
    if (!opt->density || !opt->density_m || !opt->density_v || !opt->feat || !opt->feat_m || !opt->feat_v)
        return DVGO_E_ARG;
    if (!dvgo::adam_hyper_ok(opt->beta1, opt->beta2, opt->eps, opt->t)) return DVGO_E_ARG;
    auto al16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
    if (!al16(opt->feat) || !al16(opt->feat_m) || !al16(opt->feat_v) ||
        (opt->feat_shadow_bf16 && (reinterpret_cast<uintptr_t>(opt->feat_shadow_bf16) & 7u) != 0) ||
        (opt->active && (reinterpret_cast<uintptr_t>(opt->active) & 3u) != 0))
        return DVGO_E_ARG;
    o->pd = opt->density;
    o->md = opt->density_m;
    o->vd = opt->density_v;
    o->pf = opt->feat;
    o->mf = opt->feat_m;
    o->vf = opt->feat_v;
    o->shadow = opt->feat_shadow_bf16;
    o->active = opt->active;
    o->c = dvgo::adam_coef(opt->lr, opt->beta1, opt->beta2, opt->eps, opt->t);
    return DVGO_OK;
}

// Workgroups of the fused grid Adam: a multiple of 8 (one share per XCD), no
// more than the XCD with the most chunks has steps of 64 vertices (by the
// vertices of an even share, a small grid, whose chunks do not reach all XCDs,
// was walked by an eighth of the workgroups it can use: a training step of 4096
// rays in 7^3 cells 472 us, now 189; 8192 in 11^3 282 and 189, in 23^3 151 and
// 129); 6 per compute unit (as many as its registers let be resident), 16 from
// 2^23 vertices on, where an uneven grid is dealt more evenly in smaller shares
// (6 and 16 per compute unit: 682 and 667 us for 128 rays in 255^3 cells, 1483
// and 1458 for 32768; 254 and 257 for 64 rays in 189^3, 182 and 190 for 8192 in
// 159^3).
int grid_adam_blocks(const GridArgs& g) {
    const int64_t nv = static_cast<int64_t>(g.n[0]) * g.n[1] * g.n[2], chunk = adam_chunk(g.n[1], g.n[2]);
    const int64_t nchunk = (nv + chunk - 1) / chunk;
    const int64_t per_xcd = (nchunk + 7) / 8 * (chunk / 64);
    int64_t b = static_cast<int64_t>(dvgo::device_cu_count()) * (nv < (1 << 23) ? 6 : 16) / 8;
    if (b > per_xcd) b = per_xcd;
    if (b < 1) b = 1;
    return static_cast<int>(8 * b);
}

// The preparation's arguments (mlp != NULL).
PrepArgs prep_args(const Common& cm, const dvgo_mlp* mlp, int* zero, int64_t nzero) {
    PrepArgs P;
    P.base = reinterpret_cast<float*>(cm.ws + cm.L.base);
    P.pe = reinterpret_cast<float*>(cm.ws + cm.L.pe);
    {
        PackArgs pk;
        pk.w1 = mlp->w1;
        pk.w2 = mlp->w2;
        pk.w1p = reinterpret_cast<float*>(cm.ws + cm.L.w1p);
        pk.w2p = reinterpret_cast<float*>(cm.ws + cm.L.w2p);
        pk.w1pb = reinterpret_cast<uint16_t*>(cm.ws + cm.L.w1pb);
        pk.w2pb = reinterpret_cast<uint16_t*>(cm.ws + cm.L.w2pb);
        pk.w2tpb = reinterpret_cast<uint16_t*>(cm.ws + cm.L.w2tpb);
        pk.w3 = mlp->w3;
        pk.b2 = mlp->b2;
        pk.b2p = reinterpret_cast<float*>(cm.ws + cm.L.b2p);
        pk.w3pb = reinterpret_cast<uint16_t*>(cm.ws + cm.L.w3pb);
        pk.w3tpb = reinterpret_cast<uint16_t*>(cm.ws + cm.L.w3tpb);
        pk.w1tpb = reinterpret_cast<uint16_t*>(cm.ws + cm.L.w1tpb);
        pk.bf16 = mlp->precision == DVGO_BF16;
        const bool xpe = mlp->pe_x == kMaxKX;
        pk.w1_in = xpe ? NetLayout<kMaxKX>::kIn : kIn;
        pk.w1_ns = xpe ? NetLayout<kMaxKX>::kS : kC;
        pk.w1_q = xpe ? NetLayout<kMaxKX>::kQ1 : NetLayout<0>::kQ1;
        pk.w1_s1 = xpe ? NetLayout<kMaxKX>::kS1 : NetLayout<0>::kS1;
        const int zblocks = zero ? grid_for(nzero, 256, dvgo::device_cu_count() * 4) : 0;
        P.pk = pk;
        P.rays_d = cm.sa.rays_d;
        P.B = cm.B;
        P.w1 = mlp->w1;
        P.b1 = mlp->b1;
        P.w1_in = pk.w1_in;
        P.view_col = pk.w1_ns;
        P.wide = zero && !pk.bf16 ? reinterpret_cast<int*>(cm.ws + cm.L.wide) : nullptr;   // (a call with an adjoint)
        P.pad = zero ? reinterpret_cast<float4*>(cm.ws + cm.L.rec) + 4 * cm.cap : nullptr;
        P.zero = zero;
        P.nzero = nzero;
        P.zblocks = zblocks;
        P.blocks = kPackThreads / 256 + (cm.B + kPrepRays - 1) / kPrepRays + zblocks;
    }
    return P;
}

int32_t run_prep(const Common& cm, const dvgo_mlp* mlp, hipStream_t s, int* zero = nullptr, int64_t nzero = 0) {
    if (mlp) {
        const PrepArgs P = prep_args(cm, mlp, zero, nzero);
        DVGO_LAUNCH(K_RAY_BASE, prep_kernel, dim3(P.blocks), dim3(256), 0, s, P);
        if (int32_t st = dvgo::launch_status()) return st;
    } else if (zero) {
        DVGO_LAUNCH(K_CELL_SCAN, fill_int_kernel, dim3(grid_for(nzero, 256, dvgo::device_cu_count() * 8)), dim3(256),
                    0, s, zero, nzero, 0);
        if (int32_t st = dvgo::launch_status()) return st;
    }
    return DVGO_OK;
}

GatherArgs gather_args(const Common& cm, const dvgo_field* field, const int64_t* n_kept) {
    GatherArgs ga;
    ga.sa = cm.sa;
    ga.g = cm.g;
    ga.density = field->density;
    ga.feat = field->feat;
    ga.n_kept = n_kept;
    ga.cap = cm.cap;
    ga.raw_out = reinterpret_cast<float*>(cm.ws + cm.L.raw);
    ga.feat_out = reinterpret_cast<float*>(cm.ws + cm.L.feat);
    return ga;
}

int gather_blocks(const Common& cm) { return grid_for(cm.cap, 256, dvgo::device_cu_count() * 16); }

int32_t run_density_gather(const Common& cm, const dvgo_field* field, const int64_t* n_kept, hipStream_t s) {
    if (cm.cap == 0) return DVGO_OK;
    DVGO_LAUNCH(K_GATHER, density_gather_kernel, dim3(gather_blocks(cm)), dim3(256), 0, s,
                gather_args(cm, field, n_kept));
    return dvgo::launch_status();
}

// The preparation and the gather of a render with a network, in one launch
// (the gather's workgroups first); without a network or samples, each alone.
int32_t run_prep_gather(const Common& cm, const dvgo_mlp* mlp, const dvgo_field* field, const int64_t* n_kept,
                        hipStream_t s, int* zero = nullptr, int64_t nzero = 0) {
    if (!mlp || cm.cap == 0) {
        if (int32_t st = run_prep(cm, mlp, s, zero, nzero)) return st;
        return run_density_gather(cm, field, n_kept, s);
    }
    const PrepArgs P = prep_args(cm, mlp, zero, nzero);
    const GatherArgs ga = gather_args(cm, field, n_kept);
    const int gb = gather_blocks(cm);
    const dim3 grid(static_cast<unsigned>(gb + P.blocks));
    if (field->feat_dtype == DVGO_BF16) DVGO_LAUNCH(K_GATHER, prep_gather_kernel<2>, grid, dim3(256), 0, s, P, ga, gb);
    else DVGO_LAUNCH(K_GATHER, prep_gather_kernel<1>, grid, dim3(256), 0, s, P, ga, gb);
    return dvgo::launch_status();
}

MlpArgs make_mlp_args(const Common& cm, const dvgo_mlp* mlp, const int64_t* n_kept, bool training) {
    MlpArgs ma;
    ma.sample_ray = cm.sa.sample_ray;
    ma.n_kept = n_kept;
    ma.cap = cm.cap;
    ma.w1 = mlp->w1;
    ma.w2 = mlp->w2;
    ma.b2 = mlp->precision == DVGO_BF16 ? mlp->b2 : reinterpret_cast<const float*>(cm.ws + cm.L.b2p);
    ma.w3 = mlp->w3;
    ma.b3 = mlp->b3;
    ma.base = reinterpret_cast<const float*>(cm.ws + cm.L.base);
    ma.pe = reinterpret_cast<const float*>(cm.ws + cm.L.pe);
    ma.w1p = reinterpret_cast<const float*>(cm.ws + cm.L.w1p);
    ma.w2p = reinterpret_cast<const float*>(cm.ws + cm.L.w2p);
    ma.w1pb = reinterpret_cast<const uint16_t*>(cm.ws + cm.L.w1pb);
    ma.w2pb = reinterpret_cast<const uint16_t*>(cm.ws + cm.L.w2pb);
    ma.w2tpb = reinterpret_cast<const uint16_t*>(cm.ws + cm.L.w2tpb);
    ma.w3pb = reinterpret_cast<const uint16_t*>(cm.ws + cm.L.w3pb);
    ma.w3tpb = reinterpret_cast<const uint16_t*>(cm.ws + cm.L.w3tpb);
    ma.w1tpb = reinterpret_cast<const uint16_t*>(cm.ws + cm.L.w1tpb);
    ma.feat = reinterpret_cast<float*>(cm.ws + cm.L.feat);
    ma.col = reinterpret_cast<float*>(cm.ws + cm.L.col);
    ma.partial = reinterpret_cast<float*>(cm.ws + cm.L.partial);
    ma.bf16 = mlp->precision == DVGO_BF16;
    ma.live = training && !ma.bf16 ? reinterpret_cast<uint32_t*>(cm.ws + cm.L.live) : nullptr;
    ma.wide = training && !ma.bf16 ? reinterpret_cast<int*>(cm.ws + cm.L.wide) : nullptr;
    return ma;
}

PosArgs make_pos_args(const Common& cm) {
    PosArgs pa;
    pa.rays_o = cm.sa.rays_o;
    pa.rays_d = cm.sa.rays_d;
    pa.jitter = cm.sa.jitter;
    pa.t_near = cm.sa.t_near;
    pa.sample_k = cm.sa.sample_k;
    pa.step = cm.sa.step;
    for (int i = 0; i < 3; ++i) {
        // box coordinates: centre and inverse half-extent, rounded once to float32
        pa.pe_c[i] = 0.5f * (cm.box_min[i] + cm.box_max[i]);
        pa.pe_ih[i] = 2.0f / (cm.box_max[i] - cm.box_min[i]);
    }
    return pa;
}

ComposeArgs make_compose(const Common& cm, const int32_t* perm, const int32_t* ray_offset, const int32_t* n_uniform,
                         const int64_t* n_kept, float act_shift, const float* bg, bool with_color) {
    ComposeArgs ca;
    std::memset(&ca, 0, sizeof(ca));
    ca.sa = cm.sa;
    ca.perm = perm;
    ca.ray_offset = ray_offset;
    ca.n_uniform = n_uniform;
    ca.n_kept = n_kept;
    ca.cap = cm.cap;
    ca.B = cm.B;
    ca.act_shift = act_shift;
    for (int i = 0; i < 3; ++i) ca.bg[i] = bg[i];
    ca.raw = reinterpret_cast<float*>(cm.ws + cm.L.raw);
    ca.col = reinterpret_cast<float*>(cm.ws + cm.L.col);
    ca.with_color = with_color;
    return ca;
}

int64_t cell_count_of(const dvgo_box& b) {
    return static_cast<int64_t>(b.n[0] - 1) * (b.n[1] - 1) * (b.n[2] - 1);
}

Common make_common(const dvgo_field* field, const float* rays_o, const float* rays_d, const float* jitter,
                   const float* t_near, const int32_t* sample_ray, const int32_t* sample_k, int64_t capacity,
                   int32_t B, float step, void* workspace) {
    Common cm;
    cm.sa.rays_o = rays_o;
    cm.sa.rays_d = rays_d;
    cm.sa.jitter = jitter;
    cm.sa.t_near = t_near;
    cm.sa.sample_ray = sample_ray;
    cm.sa.sample_k = sample_k;
    cm.sa.step = step;
    cm.g = dvgo::make_grid(field->box);
    for (int i = 0; i < 3; ++i) {
        cm.box_min[i] = field->box.xyz_min[i];
        cm.box_max[i] = field->box.xyz_max[i];
    }
    cm.L = ws_layout(B, capacity, cell_count_of(field->box));
    cm.ws = static_cast<char*>(workspace);
    cm.cap = capacity;
    cm.B = B;
    return cm;
}

// Binning state of a backward call inside the workspace.
struct Bins {
    int64_t ncell;
    int* cell_count;
    int* cell_start;
    int2* cell_rank;
    float4* rec_head;
    float4* rec;
};

Bins bins_of(const Common& cm, const dvgo_field* field) {
    Bins b;
    b.ncell = cell_count_of(field->box);
    b.cell_count = reinterpret_cast<int*>(cm.ws + cm.L.cell_count);
    b.cell_start = reinterpret_cast<int*>(cm.ws + cm.L.cell_start);
    b.cell_rank = reinterpret_cast<int2*>(cm.ws + cm.L.cell_rank);
    b.rec_head = reinterpret_cast<float4*>(cm.ws + cm.L.rec_head);
    b.rec = reinterpret_cast<float4*>(cm.ws + cm.L.rec);
    return b;
}

// Records placed in binned order (by the network backward, or here when
// there is none), then a lane quad per vertex: gradient into the grids, or
// the grids' fused Adam step.
int32_t run_vertex(const Common& cm, const dvgo_field* field, const Bins& b, bool with_feat, bool place,
                   const int64_t* n_kept, float* grad_density, float* grad_feat, const GridAdamArgs* opt,
                   hipStream_t s, const ReduceArgs* red = nullptr) {
    BinArgs ba;
    ba.sa = cm.sa;
    ba.g = cm.g;
    ba.n_kept = n_kept;
    ba.cap = cm.cap;
    ba.ncell = b.ncell;
    ba.cell_count = b.cell_count;
    ba.cell_start = b.cell_start;
    ba.cell_rank = b.cell_rank;
    ba.rec_head = b.rec_head;
    ba.with_feat = with_feat;
    ba.rec = b.rec;
    ba.grad_density = grad_density;
    ba.grad_feat = grad_feat;
    const int cus = dvgo::device_cu_count();
    if (place) {
        DVGO_LAUNCH(K_BIN_PLACE, bin_place_kernel, dim3(grid_for(cm.cap, 256, cus * 16)), dim3(256), 0, s, ba);
        if (int32_t st = dvgo::launch_status()) return st;
    }
    const int64_t nv = static_cast<int64_t>(field->box.n[0]) * field->box.n[1] * field->box.n[2];
    if (opt && red) {
        const int vb = grid_adam_blocks(ba.g);
        DVGO_LAUNCH(K_GRID_ADAM, vertex_adam_reduce_kernel, dim3(vb + (red->nparams + 63) / 64), dim3(256), 0, s, ba,
                    *opt, vb, *red);
    } else if (opt)
        DVGO_LAUNCH(K_GRID_ADAM, vertex_adam_kernel, dim3(grid_adam_blocks(ba.g)), dim3(256), 0, s, ba, *opt);
    else
        DVGO_LAUNCH(K_SCATTER, vertex_gather_kernel, dim3(grid_for(nv, 64, cus * 16)), dim3(256), 0, s, ba);
    return dvgo::launch_status();
}

int32_t render_bwd_impl(const dvgo_field* field, const dvgo_mlp* mlp, const float* rays_o, const float* rays_d,
                        const float* jitter, const float* t_near, const int32_t* n_uniform, const int32_t* perm,
                        const int32_t* ray_offset, const int32_t* sample_ray, const int32_t* sample_k,
                        const int64_t* n_kept, int64_t capacity, int32_t B, float step, const float* bg,
                        const float* log_t_end, const float* grad_rgb, const float* grad_depth,
                        const float* grad_acc, float* grad_density, float* grad_feat, const GridAdamArgs* opt,
                        float* grad_mlp, void* workspace, size_t workspace_bytes, void* stream,
                        bool forward_done = false, const float* sq_err = nullptr, float* loss = nullptr,
                        const NetAdam* net = nullptr, const float* aux_target = nullptr, float w_pt = 0.0f,
                        float w_bg = 0.0f, const ComposeArgs* fwd_compose = nullptr) {
    if (int32_t st = validate(field, mlp, rays_o, rays_d, t_near, n_uniform, perm, ray_offset, sample_ray, sample_k,
                              n_kept, capacity, B, step, bg, workspace, workspace_bytes))
        return st;
    if (B > 0 && (!log_t_end || (!opt && !grad_density))) return DVGO_E_ARG;
    if (mlp && ((!opt && !grad_feat) || !grad_mlp)) return DVGO_E_ARG;
    if (opt && !mlp) return DVGO_E_ARG;
    if (!mlp && grad_rgb) return DVGO_E_ARG;
    hipStream_t s = dvgo::as_stream(stream);
    if (B == 0 || capacity == 0) {
        if (!opt) return DVGO_OK;
        // no samples: every vertex still takes its zero-gradient Adam step
        BinArgs ba{};
        ba.g = dvgo::make_grid(field->box);
        DVGO_LAUNCH(K_GRID_ADAM, vertex_adam_kernel, dim3(grid_adam_blocks(ba.g)), dim3(256), 0, s, ba, *opt);
        return dvgo::launch_status();
    }
    Common cm = make_common(field, rays_o, rays_d, jitter, t_near, sample_ray, sample_k, capacity, B, step,
                            workspace);
    const Bins bins = bins_of(cm, field);
    MlpArgs ma;
    if (mlp) ma = make_mlp_args(cm, mlp, n_kept, true);
    if (!forward_done) {
        // prep (packing, per-ray encoding) also clears the cell counts
        if (int32_t st = run_prep_gather(cm, mlp, field, n_kept, s, bins.cell_count, bins.ncell + 1)) return st;
        if (mlp) {
            launch_mlp_fwd(ma, make_pos_args(cm), mlp->pe_x, dvgo::device_cu_count(), s);
            if (int32_t st = dvgo::launch_status()) return st;
        }
    }
    // adjoint of the compositing; bins every sample by fine cell on the way
    ComposeArgs ca = make_compose(cm, perm, ray_offset, n_uniform, n_kept, field->act_shift, bg, mlp != nullptr);
    ca.log_t_end_in = log_t_end;
    ca.target = aux_target;
    ca.w_pt = w_pt;
    ca.w_bg = w_bg;
    ca.grad_rgb = grad_rgb;
    ca.grad_depth = grad_depth;
    ca.grad_acc = grad_acc;
    ca.g = cm.g;
    ca.cell_count = bins.cell_count;
    ca.cell_rank = bins.cell_rank;
    ca.rec_head = bins.rec_head;
    if (mlp) ca.wide = ma.wide;
    if (fwd_compose)   // the forward compositing not yet run: both in one launch
        DVGO_LAUNCH(K_COMPOSE_BWD, compose_step_kernel, compose_grid(B), dim3(kComposeThreads), 0, s, *fwd_compose, ca);
    else
        DVGO_LAUNCH(K_COMPOSE_BWD, compose_bwd_kernel, compose_grid(B), dim3(kComposeThreads), 0, s, ca);
    if (int32_t st = dvgo::launch_status()) return st;
    if (int32_t st = run_cell_scan(bins.cell_count, bins.ncell + 1, cm.ws + cm.L.scan_tmp, bins.cell_start, s)) return st;
    int nblk = 0;
    if (mlp) {   // the network adjoint writes each sample's record at its binned position
        ma.cell_rank = bins.cell_rank;
        ma.cell_start = bins.cell_start;
        ma.rec_head = bins.rec_head;
        ma.rec = bins.rec;
        nblk = dvgo::device_cu_count();
        if (nblk > kMaxBwdBlocks) nblk = kMaxBwdBlocks;
        launch_mlp_bwd(ma, make_pos_args(cm), mlp->pe_x, nblk, s);
        if (int32_t st = dvgo::launch_status()) return st;
    }
    ReduceArgs red{};
    if (mlp) {
        red.net = NetAdam{};
        if (net) red.net = *net;
        const bool xpe = mlp->pe_x == kMaxKX;
        red.partial = reinterpret_cast<const float*>(cm.ws + cm.L.partial);
        red.nblk = nblk;
        red.nparams = xpe ? NetLayout<kMaxKX>::kParams : kMlpParams;
        red.pstride = xpe ? NetLayout<kMaxKX>::kPStride : kPStride;
        red.out = grad_mlp;
        red.sq_err = sq_err;
        red.B = B;
        red.loss = loss;
    }
    // with the fused grid Adam, the network's reduction rides in its launch
    const bool merged = mlp && opt;
    if (int32_t st = run_vertex(cm, field, bins, mlp != nullptr, mlp == nullptr, n_kept, grad_density, grad_feat, opt,
                                s, merged ? &red : nullptr))
        return st;
    if (mlp && !merged) {
        DVGO_LAUNCH(K_REDUCE, reduce_partials_kernel, dim3((red.nparams + 63) / 64), dim3(256), 0, s, red);
        if (int32_t st = dvgo::launch_status()) return st;
    }
    return DVGO_OK;
}

}  // namespace

extern "C" {

int64_t dvgo_mlp_param_count(int32_t channels, int32_t hidden, int32_t pe_x) {
    if (channels < 0 || hidden < 0 || pe_x < 0) return 0;
    const int64_t in = channels + (pe_x ? 3 + 6 * pe_x : 0) + kPE;
    return hidden * in + hidden + static_cast<int64_t>(hidden) * hidden + hidden + 3LL * hidden + 3;
}

size_t dvgo_render_workspace_bytes(int32_t B, int64_t capacity, int32_t channels, const dvgo_box* grid) {
    if (B < 0 || capacity < 0 || channels != kC || !dvgo::box_ok(grid, 2)) return 0;
    return ws_layout(B, capacity, cell_count_of(*grid)).total;
}

size_t dvgo_render_bf16_workspace_bytes(int32_t B, int64_t capacity, int32_t channels, const dvgo_box* grid) {
    if (B < 0 || capacity < 0 || channels != kC || !dvgo::box_ok(grid, 2)) return 0;
    return ws_layout(B, capacity, cell_count_of(*grid)).live;
}

// The forward uses the front of the layout only: per-ray encodings, packed
// network, per-sample density, features and colour.
size_t dvgo_render_fwd_workspace_bytes(int32_t B, int64_t capacity, int32_t channels, const dvgo_box* grid) {
    if (B < 0 || capacity < 0 || channels != kC || !dvgo::box_ok(grid, 2)) return 0;
    return ws_layout(B, capacity, cell_count_of(*grid)).partial;
}

int32_t dvgo_render_fwd(const dvgo_field* field, const dvgo_mlp* mlp, const float* rays_o, const float* rays_d,
                        const float* jitter, const float* t_near, const int32_t* n_uniform, const int32_t* perm,
                        const int32_t* ray_offset, const int32_t* sample_ray, const int32_t* sample_k,
                        const int64_t* n_kept, int64_t capacity, int32_t B, float step, const float* bg, float* rgb,
                        float* depth, float* acc, float* log_t_end, float* seg_w, float* sample_w, void* workspace,
                        size_t workspace_bytes, void* stream) {
    if (int32_t st = validate(field, mlp, rays_o, rays_d, t_near, n_uniform, perm, ray_offset, sample_ray, sample_k,
                              n_kept, capacity, B, step, bg, workspace, workspace_bytes, true))
        return st;
    if (!log_t_end && B > 0) return DVGO_E_ARG;
    if (!mlp && rgb) return DVGO_E_ARG;
    hipStream_t s = dvgo::as_stream(stream);
    if (B == 0) return DVGO_OK;
    Common cm = make_common(field, rays_o, rays_d, jitter, t_near, sample_ray, sample_k, capacity, B, step,
                            workspace);
    // with a network, the preparation and the gather first; without one
    // the compositing interpolates each sample's density itself
    if (mlp) {
        if (int32_t st = run_prep_gather(cm, mlp, field, n_kept, s)) return st;
    }
    if (mlp && capacity > 0) {
        MlpArgs ma = make_mlp_args(cm, mlp, n_kept, false);
        launch_mlp_fwd(ma, make_pos_args(cm), mlp->pe_x, dvgo::device_cu_count(), s);
        if (int32_t st = dvgo::launch_status()) return st;
    }
    ComposeArgs ca = make_compose(cm, perm, ray_offset, n_uniform, n_kept, field->act_shift, bg, mlp != nullptr);
    ca.rgb = rgb;
    ca.depth = depth;
    ca.acc = acc;
    ca.log_t_end = log_t_end;
    ca.seg_w = seg_w;
    ca.sample_w = sample_w;
    if (!mlp) {
        ca.density_in = field->density;
        ca.g = cm.g;
        DVGO_LAUNCH(K_COMPOSE_FWD, compose_fwd_kernel<true>, compose_grid(B), dim3(kComposeThreads), 0, s, ca);
    } else {
        DVGO_LAUNCH(K_COMPOSE_FWD, compose_fwd_kernel<false>, compose_grid(B), dim3(kComposeThreads), 0, s, ca);
    }
    return dvgo::launch_status();
}

int32_t dvgo_render_bwd(const dvgo_field* field, const dvgo_mlp* mlp, const float* rays_o, const float* rays_d,
                        const float* jitter, const float* t_near, const int32_t* n_uniform, const int32_t* perm,
                        const int32_t* ray_offset, const int32_t* sample_ray, const int32_t* sample_k,
                        const int64_t* n_kept, int64_t capacity, int32_t B, float step, const float* bg,
                        const float* log_t_end, const float* grad_rgb, const float* grad_depth,
                        const float* grad_acc, float* grad_density, float* grad_feat, float* grad_mlp,
                        void* workspace, size_t workspace_bytes, void* stream) {
    return render_bwd_impl(field, mlp, rays_o, rays_d, jitter, t_near, n_uniform, perm, ray_offset, sample_ray,
                           sample_k, n_kept, capacity, B, step, bg, log_t_end, grad_rgb, grad_depth, grad_acc,
                           grad_density, grad_feat, nullptr, grad_mlp, workspace, workspace_bytes, stream);
}

int32_t dvgo_grid_active_init(const float* density_m, const float* density_v, const float* feat_m,
                              const float* feat_v, int64_t n_vertices, uint32_t* active, void* stream) {
    if (n_vertices < 0) return DVGO_E_ARG;
    if (n_vertices == 0) return DVGO_OK;
    if (!density_m || !density_v || !feat_m || !feat_v || !active) return DVGO_E_ARG;
    if ((reinterpret_cast<uintptr_t>(feat_m) & 15u) || (reinterpret_cast<uintptr_t>(feat_v) & 15u) ||
        (reinterpret_cast<uintptr_t>(active) & 3u))
        return DVGO_E_ARG;
    const int64_t want = (n_vertices + 255) / 256;
    const int64_t cap = static_cast<int64_t>(dvgo::device_cu_count()) * 8;
    const int blocks = static_cast<int>(want < cap ? want : cap);
    DVGO_LAUNCH(K_GRID_ACTIVE, grid_active_kernel, dim3(blocks), dim3(256), 0, dvgo::as_stream(stream), density_m,
                density_v, feat_m, feat_v, n_vertices, active);
    return dvgo::launch_status();
}

int32_t dvgo_render_bwd_adam(const dvgo_field* field, const dvgo_mlp* mlp, const float* rays_o,
                             const float* rays_d, const float* jitter, const float* t_near, const int32_t* n_uniform,
                             const int32_t* perm, const int32_t* ray_offset, const int32_t* sample_ray,
                             const int32_t* sample_k, const int64_t* n_kept, int64_t capacity, int32_t B, float step,
                             const float* bg, const float* log_t_end, const float* grad_rgb, const float* grad_depth,
                             const float* grad_acc, const dvgo_grid_adam* opt, float* grad_mlp, void* workspace,
                             size_t workspace_bytes, void* stream) {
    if (!opt || !field) return DVGO_E_ARG;
    GridAdamArgs o;
    if (int32_t st = grid_adam_args(opt, &o)) return st;
    return render_bwd_impl(field, mlp, rays_o, rays_d, jitter, t_near, n_uniform, perm, ray_offset, sample_ray,
                           sample_k, n_kept, capacity, B, step, bg, log_t_end, grad_rgb, grad_depth, grad_acc, nullptr,
                           nullptr, &o, grad_mlp, workspace, workspace_bytes, stream);
}

int32_t dvgo_train_step(const dvgo_field* field, const dvgo_mlp* mlp, const float* rays_o, const float* rays_d,
                        const float* jitter, const float* t_near, const int32_t* n_uniform, const int32_t* perm,
                        const int32_t* ray_offset, const int32_t* sample_ray, const int32_t* sample_k,
                        const int64_t* n_kept, int64_t capacity, int32_t B, float step, const float* bg,
                        const float* target, float* rgb, float* loss, const dvgo_grid_adam* opt, float* grad_mlp,
                        const dvgo_adam_state* mlp_opt, const dvgo_aux_loss* aux, void* workspace,
                        size_t workspace_bytes, void* stream) {
    if (int32_t st = validate(field, mlp, rays_o, rays_d, t_near, n_uniform, perm, ray_offset, sample_ray, sample_k,
                              n_kept, capacity, B, step, bg, workspace, workspace_bytes))
        return st;
    if (!mlp || !opt || !grad_mlp || (B > 0 && !target)) return DVGO_E_ARG;
    const float w_pt = aux ? aux->w_pt_rgb : 0.0f, w_bg = aux ? aux->w_bg_entropy : 0.0f;
    if (!(w_pt >= 0.0f) || !(w_bg >= 0.0f)) return DVGO_E_ARG;
    NetAdam net{};
    if (mlp_opt) {
        if (!mlp_opt->param || !mlp_opt->m || !mlp_opt->v ||
            !dvgo::adam_hyper_ok(mlp_opt->beta1, mlp_opt->beta2, mlp_opt->eps, mlp_opt->t))
            return DVGO_E_ARG;
        net.param = mlp_opt->param;
        net.m = mlp_opt->m;
        net.v = mlp_opt->v;
        net.c = dvgo::adam_coef(mlp_opt->lr, mlp_opt->beta1, mlp_opt->beta2, mlp_opt->eps, mlp_opt->t);
    }
    char* ws = static_cast<char*>(workspace);
    const WsLayout L = ws_layout(B, capacity, cell_count_of(field->box));
    float* rgb_w = rgb ? rgb : reinterpret_cast<float*>(ws + L.step_rgb);
    float* grad_w = reinterpret_cast<float*>(ws + L.step_grad);
    float* logt_w = reinterpret_cast<float*>(ws + L.step_logt);
    if (B == 0 || capacity == 0) {   // nothing shared to reuse: the separate calls
        if (int32_t st = dvgo_render_fwd(field, mlp, rays_o, rays_d, jitter, t_near, n_uniform, perm, ray_offset,
                                         sample_ray, sample_k, n_kept, capacity, B, step, bg, rgb_w, nullptr,
                                         nullptr, logt_w, nullptr, nullptr, workspace, workspace_bytes, stream))
            return st;
        if (int32_t st = dvgo_photo_loss(rgb_w, target, B, grad_w, loss, stream)) return st;
        if (int32_t st = dvgo_render_bwd_adam(field, mlp, rays_o, rays_d, jitter, t_near, n_uniform, perm,
                                              ray_offset, sample_ray, sample_k, n_kept, capacity, B, step, bg, logt_w,
                                              grad_w, nullptr, nullptr, opt, grad_mlp, workspace, workspace_bytes,
                                              stream))
            return st;
        if (!mlp_opt) return DVGO_OK;
        return dvgo_adam_step(mlp_opt->param, grad_mlp, mlp_opt->m, mlp_opt->v, nullptr,
                              dvgo_mlp_param_count(field->channels, mlp->hidden, mlp->pe_x), mlp_opt->lr, mlp_opt->beta1,
                              mlp_opt->beta2, mlp_opt->eps, mlp_opt->t, stream);
    }
    GridAdamArgs o;
    if (int32_t st = grid_adam_args(opt, &o)) return st;
    hipStream_t s = dvgo::as_stream(stream);
    // forward: prep (also clears the cell counts), gather, network, compositing
    Common cm = make_common(field, rays_o, rays_d, jitter, t_near, sample_ray, sample_k, capacity, B, step,
                            workspace);
    const Bins bins = bins_of(cm, field);
    if (int32_t st = run_prep_gather(cm, mlp, field, n_kept, s, bins.cell_count, bins.ncell + 1)) return st;
    MlpArgs ma = make_mlp_args(cm, mlp, n_kept, true);
    launch_mlp_fwd(ma, make_pos_args(cm), mlp->pe_x, dvgo::device_cu_count(), s);
    if (int32_t st = dvgo::launch_status()) return st;
    float* sq_w = reinterpret_cast<float*>(ws + L.step_sqerr);
    ComposeArgs ca = make_compose(cm, perm, ray_offset, n_uniform, n_kept, field->act_shift, bg, true);
    ca.rgb = rgb_w;
    ca.log_t_end = logt_w;
    ca.target = target;          // the loss gradient comes out of the compositing
    ca.grad_rgb_out = grad_w;
    ca.sq_err = sq_w;
    ca.w_pt = w_pt;
    ca.w_bg = w_bg;
    // adjoint and Adam, reusing the forward's gathered features, colours and
    // prep; the compositing (ca) runs in the adjoint's first launch
    return render_bwd_impl(field, mlp, rays_o, rays_d, jitter, t_near, n_uniform, perm, ray_offset, sample_ray,
                           sample_k, n_kept, capacity, B, step, bg, logt_w, grad_w, nullptr, nullptr, nullptr,
                           nullptr, &o, grad_mlp, workspace, workspace_bytes, stream, true, sq_w, loss,
                           mlp_opt ? &net : nullptr, target, w_pt, w_bg, &ca);
}

}  // extern "C"
