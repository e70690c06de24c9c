// Monarch layers in full precision (fp32) with few tokens or narrow blocks, both batched products in ONE kernel on
// the fp32 matrix instructions (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation).
//
// What bounds it: latency. The layers that run in fp32 are small (256 ... 1024 wide, some tokens), their factors fit
// every L2, and the portable kernel walked them in serial steps of 16 contraction indices with a global load, two
// barriers and 4-byte LDS traffic in each, on four workgroups (256 x 256, 4 blocks, 8 tokens: 9.0 us per product, two
// of them). Here a call is one launch that every compute unit enters with its weights already on the way.
//
// Workgroup = 16 tokens x one output block k x a range of its outputs:
//   phase 0  X[16][n_in] -> LDS (rows past T repeat the last row and are never stored)
//   phase 1  Z'_k[t][l r' + rho] = sum_a X[t][l p + a] R[l][rho b2 + k][a]   -> LDS
//   phase 2  Y[t][o(k, j)] = sum_m Z'_k[t][m] L[k][j][m]                     -> global
// The weight rows are the first operand, 16 of them per tile, straight from global memory as 16-byte loads (four
// lanes on 64 contiguous bytes of a row; component c of lane (row, g) is contraction index 4 g + c of the 16, the same
// in both operands). Accumulator element e of a lane is output column 4 (lane / 16) + e of token lane % 16.
// A wavefront takes every nw-th tile of a phase, 64 contraction indices (an item) at a time; the first item of phase 2
// is requested at the start (the weights depend on nothing). At these sizes the instructions are data too: code that
// runs once per launch is fetched at the latency of the L2, so the loops are rolled and there is no division, and a
// software pipeline is only worth its code where a wavefront has several items (256 x 256, 4 blocks, 8 tokens: 8.6 us
// with four unrolled buffers per phase, 18 KB of code, 4.9 with three, 4.4 with one; 18.1 on the portable kernel.
// 1024 x 1024: 16.6 with three buffers, 49 on the portable kernel).
#include "blr_common.h"

namespace blr {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int FM_TT = 16;            // tokens per workgroup

struct MonarchF32Args {
    const float *X, *R, *L;
    float* Y;
    int64_t T;
    int n_in, n_out, b1, b2, rp, p, q, w2;
    int tpl;                         // 16-row tiles of one input block's rank indices
    int qt;                          // outputs per workgroup (a multiple of 16)
    int out_step, out_block;         // output j of block k is element k out_block + j out_step of its row
    int xstr, zstr;                  // LDS row strides in floats
};

// DEEP: two items in flight behind the one in use, in three register buffers; else one item at a time (a wavefront has
// about one per phase)
template <bool DEEP>
__global__ __launch_bounds__(512) void monarch_f32_kernel(MonarchF32Args a) {
    extern __shared__ __attribute__((aligned(16))) float sm[];
    float* Xs = sm;                                     // [16][xstr]
    float* Zs = sm + FM_TT * a.xstr;                    // [16][zstr]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int l16 = lane & 15, kg = lane >> 4;
    const int k = blockIdx.x, j0 = blockIdx.y * a.qt;
    const int64_t t0 = (int64_t)blockIdx.z * FM_TT;
    const int nj = a.q - j0 < a.qt ? a.q - j0 : a.qt;

    // One phase: rows 16 sub + ... of block l of the weights, whose row pitch is `pitch`; nl blocks of `rows` rows
    struct Phase {
        const float* weights;
        int64_t pitch;
        int nl, tpl, rows, K;
    };
    struct Cursor { int l, sub, k0; };                  // block, tile in it, first contraction index of the item (uniform)
    auto settle = [&](const Phase& ph, Cursor& c) {
        while (c.sub >= ph.tpl) { c.sub -= ph.tpl; ++c.l; }
    };
    auto next = [&](const Phase& ph, Cursor& c) {
        c.k0 += 64;
        if (c.k0 >= ph.K) {
            c.k0 = 0;
            c.sub += nw;
            settle(ph, c);
        }
    };
    auto fetch = [&](const Phase& ph, const Cursor& c, f32x4 (&w)[4]) {
        if (c.l >= ph.nl) return;                       // uniform
        int row = c.sub * 16 + l16;
        row = row < ph.rows ? row : ph.rows - 1;        // rows past the block: never stored
        const float* src = ph.weights + ((int64_t)c.l * ph.rows + row) * ph.pitch;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int kk = c.k0 + u * 16 + kg * 4;
            w[u] = *(const f32x4*)(src + (kk < ph.K ? kk : ph.K - 4));    // past K: re-read, zeroed on use
        }
    };
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;     // (two chains of dependent MFMAs)
    auto multiply = [&](const Phase& ph, const Cursor& c, const float* tok, const f32x4 (&w)[4]) {
        if (c.k0 + 64 <= ph.K) {                        // uniform: a whole item needs no selects (256 x 256, 8 tokens: 4.2 -> 3.9 us; 1024 x 1024: 16.5 -> 15.5)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const f32x4 x = *(const f32x4*)(tok + c.k0 + u * 16 + kg * 4);
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][e], x[e], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][e + 1], x[e + 1], acc1, 0, 0, 0);
                }
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {                   // past K both operands are zero (an infinity times zero would be NaN)
            const int kk = c.k0 + u * 16 + kg * 4;
            const bool in = kk < ph.K;
            const f32x4 x = *(const f32x4*)(tok + (in ? kk : ph.K - 4));
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? w[u][e] : 0.f, in ? x[e] : 0.f, acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? w[u][e + 1] : 0.f, in ? x[e + 1] : 0.f, acc1, 0, 0, 0);
            }
        }
    };
    // every item of a phase: multiplied with its part of this lane's token; done(l, first row of the lane, sum) per tile.
    auto run = [&](const Phase& ph, Cursor c, const float* tok, int tok_block, f32x4 (&w)[4], auto done) {
        auto use = [&](const f32x4 (&v)[4]) {
            multiply(ph, c, tok + c.l * tok_block, v);
            const int l = c.l, sub = c.sub;
            next(ph, c);
            if (c.k0 == 0) {
                done(l, sub * 16 + 4 * kg, acc0 + acc1);
                acc0 = acc1 = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        };
        if constexpr (DEEP) {
            f32x4 wa[4], wb[4];
            Cursor f = c;
            auto item = [&](const f32x4 (&v)[4], f32x4 (&load)[4]) {
                next(ph, f);
                fetch(ph, f, load);
                if (c.l < ph.nl) use(v);                // uniform
            };
            next(ph, f);
            fetch(ph, f, wa);
#pragma unroll 1
            while (c.l < ph.nl) {                       // uniform
                item(w, wb);
                item(wa, w);
                item(wb, wa);
            }
        } else {
#pragma unroll 1
            while (c.l < ph.nl) {                       // uniform
                use(w);
                fetch(ph, c, w);
            }
        }
    };

    const Phase p1{a.R + (int64_t)k * a.p, (int64_t)a.b2 * a.p, a.b1, a.tpl, a.rp, a.p};
    const Phase p2{a.L + ((int64_t)k * a.q + j0) * a.w2, a.w2, 1, (nj + 15) >> 4, nj, a.w2};
    Cursor c1{0, wave, 0}, c2{0, wave, 0};
    settle(p1, c1);
    settle(p2, c2);
    f32x4 w1[4], w2[4];
    fetch(p1, c1, w1);
    {                                                   // X tile: a wavefront moves whole rows, four loads in flight
        const int pieces = a.n_in >> 2, last = a.T - t0 > FM_TT ? FM_TT - 1 : (int)(a.T - t0) - 1;
        const int row = tid >> 5;                       // 32 lanes per row; all 16 rows at once with 8 wavefronts, 8 with 4
#pragma unroll 1
        for (int r0 = row; r0 < FM_TT; r0 += nw * 2) {
            const float* xt = a.X + (t0 + (r0 < last ? r0 : last)) * a.n_in;
#pragma unroll 1
            for (int c0 = tid & 31; c0 < pieces; c0 += 128) {
                f32x4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = *(const f32x4*)(xt + (c0 + u * 32 < pieces ? c0 + u * 32 : c0) * 4);
#pragma unroll
                for (int u = 0; u < 4; ++u) *(f32x4*)(Xs + r0 * a.xstr + (c0 + u * 32 < pieces ? c0 + u * 32 : c0) * 4) = v[u];
            }
        }
    }
    fetch(p2, c2, w2);
    __syncthreads();
    run(p1, c1, Xs + l16 * a.xstr, a.p, w1, [&](int l, int row, f32x4 v) {
        if (row < a.rp) *(f32x4*)(Zs + l16 * a.zstr + l * a.rp + row) = v;
    });
    __syncthreads();                                    // Z'_k is complete
    const bool live = t0 + l16 < a.T;
    float* y = a.Y + (t0 + l16) * a.n_out + (int64_t)k * a.out_block + (int64_t)j0 * a.out_step;
    run(p2, c2, Zs + l16 * a.zstr, 0, w2, [&](int, int row, f32x4 v) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (live && row + e < nj) y[(int64_t)(row + e) * a.out_step] = v[e];
    });
}

// Output ranges per block: only while the launch has idle compute units and every wavefront keeps a tile (each range
// computes Z'_k again).
inline void choose_ranges(int64_t T, int b2, int q, int& jsplit, int& qt) {
    const int64_t base = ((T + FM_TT - 1) / FM_TT) * b2;
    const int tiles = (q + 15) / 16;
    int s = base >= 256 ? 1 : (int)(256 / base);
    if (s > tiles / 8) s = tiles / 8;
    if (s < 1) s = 1;
    qt = ((tiles + s - 1) / s) * 16;
    jsplit = (q + qt - 1) / qt;
}

inline int64_t lds_bytes(int n_in, int w2) { return (int64_t)FM_TT * ((n_in + 4) + (w2 + 4)) * 4; }

template <bool DEEP>
hipError_t launch_inst(const MonarchF32Args& a, dim3 grid, dim3 block, int lds, hipStream_t s) {
    static LdsLimitOnce lds_limit;
    if (hipError_t e = lds_limit.set({(const void*)monarch_f32_kernel<DEEP>}, 160 * 1024); e != hipSuccess) return e;
    hipLaunchKernelGGL(monarch_f32_kernel<DEEP>, grid, block, lds, s, a);
    return hipGetLastError();
}

}  // namespace

bool monarch_f32_supported(int64_t T, int n_in, int n_out, int b1, int b2, int rp) {
    if (T <= 0 || b1 <= 0 || b2 <= 0 || rp <= 0 || n_in % b1 || n_out % b2) return false;
    const int p = n_in / b1;
    const int64_t w2 = (int64_t)b1 * rp;
    if (p % 4 || rp % 4 || w2 > 8192 || n_in > 8192) return false;            // 16-byte rows of both factors, 16-byte pieces of Z'
    if ((T + FM_TT - 1) / FM_TT > 65535) return false;                       // grid.z
    return lds_bytes(n_in, (int)w2) <= 160 * 1024;
}

hipError_t launch_monarch_f32(const void* X, const void* R, const void* L, void* Y, int64_t T, int n_in, int n_out,
                              int b1, int b2, int rp, bool out_blocked, hipStream_t s) {
    MonarchF32Args a{};
    a.X = (const float*)X; a.R = (const float*)R; a.L = (const float*)L; a.Y = (float*)Y;
    a.T = T; a.n_in = n_in; a.n_out = n_out; a.b1 = b1; a.b2 = b2; a.rp = rp;
    a.p = n_in / b1; a.q = n_out / b2; a.w2 = b1 * rp;
    a.tpl = (rp + 15) / 16;
    int jsplit;
    choose_ranges(T, b2, a.q, jsplit, a.qt);
    a.out_step = out_blocked ? 1 : b2; a.out_block = out_blocked ? a.q : 1;
    a.xstr = n_in + 4; a.zstr = a.w2 + 4;
    const int K = a.p > a.w2 ? a.p : a.w2;
    // as many wavefronts as the wider phase has tiles, 4 or 8
    const int tiles = b1 * a.tpl > a.qt / 16 ? b1 * a.tpl : a.qt / 16;
    const dim3 grid((unsigned)b2, (unsigned)jsplit, (unsigned)((T + FM_TT - 1) / FM_TT)), block(tiles <= 4 ? 256 : 512);
    const int lds = (int)lds_bytes(n_in, a.w2);
    return K <= 64 && tiles <= 8 ? launch_inst<false>(a, grid, block, lds, s) : launch_inst<true>(a, grid, block, lds, s);
}

}  // namespace blr
