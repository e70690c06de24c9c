// bf16 MFMA batched "NT" GEMM for FEW tokens (M <= 32): the weight-streaming regime. Also used tile by tile (32 tokens
// per workgroup) for products with small weights, few 64 x 64 tiles and a long contraction index, where the weights
// then come from L2.
//
// With few tokens the product is a stream of the weights through the chip, so the tiling is turned around: a
// workgroup owns 16 weight rows (output columns) and ALL tokens, and its wavefronts split the contraction index
// between them (split-K inside the workgroup, summed through LDS in wavefront order, so results do not depend on
// timing). Many small workgroups (N/16 per batch entry) put every compute unit to work on the stream.
//
// What bounds it: a launch (1.6 us for an empty kernel in a graph) plus one memory latency, and the instructions
// themselves: code that runs once per launch is fetched at the latency of the L2. So the loops are rolled, the operands
// go to LDS with direct loads (no registers, hence no unrolling, to hold what is in flight), and the index maps are
// grid dimensions instead of divisions. Monarch 4096 x 4096, 4 blocks, r = 1024, both products with weights from the
// memory-side cache (16.8 MB): 6.8 us for one token and 7.5 for 16, against 9.1 and 9.9 with eight unrolled register
// buffers, cross-lane permutes and a general column map per element.
//
// The weight fragment is the first MFMA operand: an accumulator lane holds four consecutive output columns of one token.
//
// For a handful of tokens the RMS normalisation in front of a product is cheaper inside it than as a launch: every workgroup
// computes the rows it multiplies (or the slice of them that its batch entry reads) into LDS while its weights are on the
// way (SkinnySource: a residual stream to which the previous linear's output is added first). The elementwise steps behind
// a group of products (the scaled sum of three, the SiLU gate) are combined where the products are: in front of the next
// one every workgroup would repeat them.
#include "skinny_source.h"

namespace blr {
namespace {

constexpr int SK_BN = 16;             // weight rows per workgroup
constexpr int SK_RD = 8;              // k32 steps in flight per wavefront

// C(g, m, s, i) = sum_k A(g, m, k) B(g, s, i, k) over segments s of n columns i each: both index maps of a GemmDesc
// (row gather of B, column scatter of C) are products of the segment and the place in it.
struct SkinnyArgs {
    const bf16_t *A, *B;
    bf16_t* C;
    int64_t a_gs, a_rs, b_gs, c_gs, c_rs, b_s, c_s, c_i;
    unsigned b_i;                     // row pitch of B inside a segment (elements)
    int M, n, K;
    int nall;                         // PACK: columns of all segments
    int a_seg;
    int64_t a_seg_stride;
    int kper;                         // contraction indices per wavefront, a multiple of 32
    int slots;                        // steps a wavefront's part of LDS holds (<= SK_RD)
    int mtiles;                       // tiles of 16 MT tokens
    int64_t a_ms, b_ms;               // MEM: distance of the members' operands
    int c_seg;                        // MEM: columns in runs of so many, c_s apart (0: one run)
    float scale;
};

// MT: 16-token tiles (M <= 16 MT); NW: wavefronts; TAIL: K is no multiple of 32
// ROWS: every wavefront owns 16 weight rows and the whole contraction index instead of a part of it (computed rows only:
// the rows serve 16 NW outputs then, and there are no partial sums to add)
// PACK: a workgroup's 16 weight rows run across segments shorter than 16
// MEM: that many products of one shape, each on NW / MEM of the wavefronts, are rounded to storage and combined: 3, their
// scaled sum; 2, SiLU(first) * second
template <int MT, int NW, bool TAIL, int SRC, bool ROWS, bool PACK, int MEM>
__global__ __launch_bounds__(64 * NW) void gemm_skinny_kernel(SkinnyArgs a, SkinnySource src) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int XL = SRC == kSrcInput ? MT : 0;        // token rows that come as direct loads, per step
    constexpr int SLOT = (1 + XL) * 1024;                // 16 weight rows and 16 XL token rows of 64 bytes
    constexpr int WPM = NW / MEM, RD = MEM > 1 ? SK_RD / 2 : SK_RD;   // wavefronts and steps in flight of a product
    static_assert(SRC == kSrcInput ? !ROWS : MT == 1 && !PACK && MEM == 1, "computed rows: a handful of tokens");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = (ROWS ? blockIdx.x * NW + wave : blockIdx.x) * SK_BN, s = blockIdx.y;
    int g = blockIdx.z, m_base = 0;
    if (a.mtiles > 1) {
        m_base = (g % a.mtiles) * (MT * 16);
        g /= a.mtiles;
    }
    // A direct load fills 16 rows of 64 bytes: lane l brings the piece of slot l % 4 of row l / 4. The pieces are
    // XOR-swizzled by the row so that the 16 rows a fragment read serves per clock cover all banks.
    const int lrow = lane >> 2, piece = (lane & 3) ^ ((lrow >> 2) & 3);
    const int member = MEM > 1 ? wave / WPM : 0, kw = ROWS ? 0 : (wave - member * WPM) * a.kper;
    const unsigned char* B = (const unsigned char*)(a.B + g * a.b_gs + s * a.b_s + (MEM > 1 ? member * a.b_ms : 0));
    const unsigned char* A = (const unsigned char*)(a.A + g * a.a_gs + m_base * a.a_rs + (MEM > 1 ? member * a.a_ms : 0));
    const int rows_n = PACK ? a.nall : a.n, row = i0 + lrow < rows_n ? i0 + lrow : rows_n - 1;   // rows past the segment repeat its last one; never stored
    unsigned woff = PACK ? (unsigned)(row % a.n) * a.b_i + (unsigned)(row / a.n) * (unsigned)a.b_s : (unsigned)row * a.b_i, xoff[MT];
#pragma unroll
    for (int mt = 0; mt < XL; ++mt) {
        const int m = mt * 16 + lrow, left = a.M - m_base - 1;
        xoff[mt] = (unsigned)(m < left ? m : left) * (unsigned)a.a_rs;
    }
    unsigned char* mine = smem + wave * (a.slots * SLOT);
    const int steps = a.K - kw <= 0 ? 0 : ((a.K - kw < a.kper ? a.K - kw : a.kper) + 31) >> 5;
    int kf = kw;                                        // contraction index under the fetch cursor
    int64_t seg_off = 0;                                // segmented contraction index of A: what to add to it (a step lies in one segment)
    int seg_left = 0x7fffffff;
    if (XL && a.a_seg) {
        seg_off = (int64_t)(kw / a.a_seg) * (a.a_seg_stride - a.a_seg);
        seg_left = a.a_seg - kw % a.a_seg;
    }
    auto fetch = [&](unsigned char* slot) {
        const unsigned kl = kf + piece * 8;
        // pieces past K are zeros in both operands (an infinity times zero would be NaN)
        auto from = [&](const unsigned char* p) { return TAIL && kl >= (unsigned)a.K ? zero_piece : p; };
        __builtin_amdgcn_global_load_lds(BLR_GPTR(from(B + (woff + kl) * 2u)), BLR_LPTR(slot), 16, 0, 0);
        const unsigned char* As = A + seg_off * 2;
#pragma unroll
        for (int mt = 0; mt < XL; ++mt)
            __builtin_amdgcn_global_load_lds(BLR_GPTR(from(As + (xoff[mt] + kl) * 2u)), BLR_LPTR(slot + (1 + mt) * 1024), 16, 0, 0);
        kf += 32;
        seg_left -= 32;
        if (XL && seg_left == 0) {
            seg_left = a.a_seg;
            seg_off += a.a_seg_stride - a.a_seg;
        }
    };
    const int l16 = lane & 15, kg = lane >> 4;
    const unsigned frag = (unsigned)(uintptr_t)BLR_LPTR(mine) + l16 * 64 + ((kg ^ ((l16 >> 2) & 3)) * 16);
    // computed rows lie behind the wavefronts' slots
    const unsigned xs = a.K * 2 + 16;
    unsigned char* rows = smem + NW * (a.slots * SLOT);
    const unsigned row_frag = (unsigned)(uintptr_t)BLR_LPTR(rows) + (l16 < a.M ? l16 : a.M - 1) * xs;
    auto x_frag = [&](int mt, unsigned at, int t) {      // token fragment of step t, whose slot is at
        if constexpr (SRC == kSrcInput) return lds_read_frag(frag + at + (1 + mt) * 1024);
        int k = kw + t * 32 + kg * 8;
        if (TAIL) k = k < a.K ? k : a.K;                 // (zeros behind the row)
        return lds_read_frag(row_frag + k * 2);
    };
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](bf16x8 w, const bf16x8 (&x)[MT]) {           // (after the wait for both)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[mt], acc[mt], 0, 0, 0);
    };

    int t = 0;
    for (; t < steps && t < a.slots; ++t) fetch(mine + t * SLOT);
    if constexpr (SRC != kSrcInput) {
        if (TAIL && tid < a.M) *(u32x4*)(rows + tid * xs + a.K * 2) = u32x4{0u, 0u, 0u, 0u};
        source_rows<SRC, NW>(src, a.M, a.K, g, rows, xs, (float*)(rows + a.M * xs));
        __syncthreads();
    }
    t = 0;
    unsigned at = 0;                                    // slot of step t (bytes)
#pragma unroll 1
    for (; t + RD < steps; ++t) {                    // (only with all RD slots: what is in flight is a constant)
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"((1 + XL) * (RD - 1)) : "memory");
        bf16x8 w = lds_read_frag(frag + at), x[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) x[mt] = x_frag(mt, at, t);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w) :: "memory");
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) asm volatile("" : "+v"(x[mt]));
        fetch(mine + at);
        multiply(w, x);
        at = at == (RD - 1) * SLOT ? 0 : at + SLOT;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
    while (t < steps) {                                 // what is left has landed; two steps per trip share an LDS latency
        const unsigned at1 = at == (unsigned)(a.slots - 1) * SLOT ? 0 : at + SLOT;
        bf16x8 w0 = lds_read_frag(frag + at), w1 = lds_read_frag(frag + at1), x0[MT], x1[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            x0[mt] = x_frag(mt, at, t);
            x1[mt] = x_frag(mt, at1, t + 1 < steps ? t + 1 : t);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w0), "+v"(w1) :: "memory");
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) asm volatile("" : "+v"(x0[mt]), "+v"(x1[mt]));
        multiply(w0, x0);
        if (t + 1 < steps) multiply(w1, x1);            // uniform
        t += 2;
        at = at1 == (unsigned)(a.slots - 1) * SLOT ? 0 : at1 + SLOT;
    }
    if constexpr (ROWS) {                               // acc[e]: token l16, column 4*kg + e
        if (l16 < a.M)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = i0 + 4 * kg + e;
                if (c < a.n) a.C[l16 * a.c_rs + g * a.c_gs + s * a.c_s + c * a.c_i] = float_to_bf16(acc[0][e]);
            }
        return;
    }
    __syncthreads();                                    // every wavefront is past its operands: the partial sums take their place

    // acc[mt][e]: token mt*16 + l16, column 4*kg + e
    float* part = (float*)smem;                         // [wave][16 MT tokens][16 columns + 4]
    constexpr int PSTR = SK_BN + 4;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
        *(f32x4*)(part + ((wave * MT + mt) * 16 + l16) * PSTR + 4 * kg) = acc[mt];
    __syncthreads();
    const int c = tid & 15, ci = i0 + c;                // (64 NW is a multiple of 16: a thread keeps its column)
    bf16_t* Cc = a.C + g * a.c_gs + (PACK ? (ci / a.n) * a.c_s + (ci % a.n) * a.c_i : MEM > 1 && a.c_seg ? (ci / a.c_seg) * a.c_s + ci % a.c_seg : s * a.c_s + ci * a.c_i);
    for (int o = tid; o < MT * 256; o += 64 * NW) {
        const int m = o >> 4;
        if (m_base + m >= a.M || ci >= rows_n) continue;
        float v[MEM];
#pragma unroll
        for (int e = 0; e < MEM; ++e) {
            v[e] = part[(e * WPM * MT * 16 + m) * PSTR + c];
#pragma unroll
            for (int w = 1; w < WPM; ++w) v[e] += part[((e * WPM + w) * MT * 16 + m) * PSTR + c];
            if (MEM > 1) v[e] = bf16_to_float(float_to_bf16(v[e]));
        }
        if constexpr (MEM == 3) v[0] = (v[0] + v[1] + v[2]) * a.scale;
        if constexpr (MEM == 2) v[0] = silu(v[0]) * v[1];
        Cc[(m_base + m) * a.c_rs] = float_to_bf16(v[0]);
    }
}

template <int MT, int NW, int SRC, bool ROWS = false, bool PACK = false, int MEM = 1>
hipError_t launch_skinny(SkinnyArgs& a, const SkinnySource& src, dim3 grid, hipStream_t s) {
    constexpr int SLOT = (1 + (SRC == kSrcInput ? MT : 0)) * 1024;
    const int nk = (a.K + 31) / 32, per = ROWS ? nk : (nk + NW / MEM - 1) / (NW / MEM), rd = MEM > 1 ? SK_RD / 2 : SK_RD;
    a.kper = per * 32;
    a.slots = per < rd ? per : rd;
    const int operands = NW * a.slots * SLOT, sums = ROWS ? 0 : NW * MT * 16 * (SK_BN + 4) * 4;
    int lds = operands;
    if (SRC != kSrcInput) lds += a.M * (a.K * 2 + 16) + a.M * 8 * 4;
    if (lds < sums) lds = sums;
    static LdsLimitOnce lds_limit;
    if (hipError_t e = lds_limit.set({(const void*)gemm_skinny_kernel<MT, NW, false, SRC, ROWS, PACK, MEM>, (const void*)gemm_skinny_kernel<MT, NW, true, SRC, ROWS, PACK, MEM>}, 160 * 1024); e != hipSuccess) return e;
    if (a.K % 32) hipLaunchKernelGGL((gemm_skinny_kernel<MT, NW, true, SRC, ROWS, PACK, MEM>), grid, dim3(64 * NW), lds, s, a, src);
    else hipLaunchKernelGGL((gemm_skinny_kernel<MT, NW, false, SRC, ROWS, PACK, MEM>), grid, dim3(64 * NW), lds, s, a, src);
    return hipGetLastError();
}

// segments of the two index maps: the whole N without a gather, else the blocks of b_div columns
inline bool segments(const GemmDesc& d, int& n, int& nseg) {
    if (d.b_div == 0 && d.c_div == 1) { n = d.N; nseg = 1; return true; }
    if (d.b_div <= 0 || d.b_div != d.c_div || d.N % d.b_div) return false;
    n = d.b_div; nseg = d.N / d.b_div;
    return nseg <= 65535;
}

bool shape_ok(const GemmDesc& d, int64_t mtiles) {
    int n, nseg;
    return segments(d, n, nseg) && mtiles * d.G <= 65535;
}

}  // namespace

bool skinny_gemm_supported(const GemmDesc& d) { return d.M <= 32 && shape_ok(d, 1); }

static SkinnyArgs skinny_args(const GemmDesc& d) {
    SkinnyArgs a{};
    int nseg;
    segments(d, a.n, nseg);
    a.A = (const bf16_t*)d.A; a.B = (const bf16_t*)d.B; a.C = (bf16_t*)d.C;
    a.a_gs = d.a_gs; a.a_rs = d.a_rs; a.b_gs = d.b_gs; a.c_gs = d.c_gs; a.c_rs = d.c_rs;
    a.M = (int)d.M; a.K = d.K;
    if (d.b_div) { a.b_i = (unsigned)(d.b_mul * d.b_rs); a.b_s = d.b_rs; a.c_i = d.c_lo; a.c_s = d.c_hi; }
    else { a.b_i = (unsigned)d.b_rs; a.b_s = 0; a.c_i = d.c_hi; a.c_s = 0; }
    a.a_seg = d.a_seg; a.a_seg_stride = d.a_seg_stride;
    a.mtiles = 1;
    return a;
}

// eight wavefronts where each still gets two or more steps: twice the bytes in flight of a workgroup and half its steps
static bool eight_waves(int K) { return K >= 512; }

// Segments of up to 8 columns leave half and more of a workgroup's 16 weight rows unused: they are packed, at a division per
// thread, from two workgroups per compute unit on (first Monarch products at 1 / 32 tokens, whole calls, packed against one
// segment per workgroup: 4096 x 4096, 128 blocks, r' = 1: 5.2 / 8.3 against 14.7 / 19.5 us; 64 blocks, r' = 4: 5.3 / 7.6 against
// 7.2 / 10.3; 32 blocks, r' = 8: 5.0 / 7.0 against 5.4 / 7.4. Below, and with 12 columns, level or 3 % behind: 2048 x 2048,
// 16 blocks, r' = 4: 4.6 / 5.6 against 4.5 / 5.4).
static bool packs(const GemmDesc& d, int n, int nseg, int64_t mtiles) { return n <= SK_BN / 2 && (int64_t)nseg * d.G * mtiles > 512; }

int64_t skinny_workgroups(const GemmDesc& d) {
    int n = 0, nseg = 0;
    segments(d, n, nseg);
    const int64_t mtiles = (d.M + 31) / 32;
    return packs(d, n, nseg, mtiles) ? (int64_t)((d.N + SK_BN - 1) / SK_BN) * d.G * mtiles : (int64_t)((n + SK_BN - 1) / SK_BN) * nseg * d.G * mtiles;
}

template <bool PACK>
static hipError_t launch_input(SkinnyArgs& a, dim3 grid, hipStream_t s) {
    if (a.M > 16) return launch_skinny<2, 4, kSrcInput, false, PACK>(a, {}, grid, s);
    return eight_waves(a.K) ? launch_skinny<1, 8, kSrcInput, false, PACK>(a, {}, grid, s) : launch_skinny<1, 4, kSrcInput, false, PACK>(a, {}, grid, s);
}

hipError_t launch_gemm_skinny(const GemmDesc& d, hipStream_t s) {
    SkinnyArgs a = skinny_args(d);
    const int mt = d.M <= 16 ? 1 : 2;                   // more than 32 tokens: one workgroup per 32-token tile and 16 weight rows
    a.mtiles = (int)((d.M + mt * 16 - 1) / (mt * 16));
    const int nseg = d.b_div ? d.N / d.b_div : 1;
    a.nall = d.N;
    if (packs(d, a.n, nseg, a.mtiles)) return launch_input<true>(a, dim3((unsigned)((d.N + SK_BN - 1) / SK_BN), 1u, (unsigned)(d.G * a.mtiles)), s);
    return launch_input<false>(a, dim3((unsigned)((a.n + SK_BN - 1) / SK_BN), (unsigned)nseg, (unsigned)(d.G * a.mtiles)), s);
}

bool gemm_combine_supported(const GemmDesc& d, int members) {
    if (d.M > 32) return gemm_members_supported(d, members);
    return d.b_div == 0 && (d.c_div == 1 || d.c_lo == 1) && d.G <= 65535 && mfma_gemm_supported(d);
}
hipError_t launch_gemm_combine(const GemmDesc& d, int members, const Combine& c, hipStream_t s) {
    if (d.M > 32) return launch_gemm_members(d, members, c, s);
    SkinnyArgs a = skinny_args(d);
    a.n = d.N;
    a.a_ms = c.a_ms; a.b_ms = c.b_ms; a.scale = c.scale;
    if (d.c_div > 1) { a.c_seg = d.c_div; a.c_s = d.c_hi; }
    const dim3 grid((unsigned)((a.n + SK_BN - 1) / SK_BN), 1u, (unsigned)d.G);
    if (members == 3) return a.M > 16 ? launch_skinny<2, 12, kSrcInput, false, false, 3>(a, {}, grid, s) : launch_skinny<1, 12, kSrcInput, false, false, 3>(a, {}, grid, s);
    return a.M > 16 ? launch_skinny<2, 8, kSrcInput, false, false, 2>(a, {}, grid, s) : launch_skinny<1, 8, kSrcInput, false, false, 2>(a, {}, grid, s);
}

bool skinny_source_supported(const GemmDesc& d) {
    return d.M >= 1 && d.M <= kSourceTokens && mfma_gemm_supported(d) && shape_ok(d, 1) && d.K <= 4096;      // (rows of 8 tokens: 64 KB of LDS behind the weights)
}

// From this many 16-row tiles on a wavefront owns a tile: there are workgroups enough, and the norm is computed a quarter as often.
// A Monarch chain layer at 1 / 2 / 3 tokens, owned against four or eight wavefronts to a tile: 4096 / 8192 in 16 blocks, r = 1024 (3072 and 2048
// tiles) 52.9 / 56.1 / 59.8 against 55.3 / 60.6 / 65.6 us; 2048 / 8192 in 16 blocks, r = 512 (1536 and 1024) 34.2 / 36.1 / 38.0 against 34.1 / 36.0 /
// 38.3; in 8 blocks, r = 1024 (the same) 45.1 / 47.1 / 49.1 against 44.6 / 46.7 / 49.1; 4096 / 8192 in 4 blocks, r = 1024 and 1536 (768 each)
// 63.1 / 66.6 / 70.2 against 61.6 / 64.3 / 67.1.
constexpr int64_t kRowsTiles = 2048;

hipError_t launch_gemm_skinny_norm(const GemmDesc& d, const SkinnySource& src, hipStream_t s) {
    SkinnyArgs a = skinny_args(d);
    const unsigned tiles = (unsigned)((a.n + SK_BN - 1) / SK_BN), nseg = d.b_div ? d.N / d.b_div : 1;
    if ((int64_t)tiles * nseg * d.G >= kRowsTiles) return launch_skinny<1, 4, kSrcNorm, true>(a, src, dim3((tiles + 3) / 4, nseg, (unsigned)d.G), s);
    const dim3 grid(tiles, nseg, (unsigned)d.G);
    return eight_waves(d.K) ? launch_skinny<1, 8, kSrcNorm>(a, src, grid, s) : launch_skinny<1, 4, kSrcNorm>(a, src, grid, s);
}

bool skinny_gemm_tiled_supported(const GemmDesc& d) { return d.M < (1ll << 20) && shape_ok(d, (d.M + 31) / 32); }

}  // namespace blr
