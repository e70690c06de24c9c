// BLAST stage 1 and coupling in one launch for FEW tokens (bf16 MFMA, gfx950): the weight-streaming counterpart of
// blast_stage12_kernel.
//
//   Z[t][j][rho] = sum_c X[t][j q + c] Vt[j][rho][c]          (rounded to bf16, on chip)
//   A[t][i][rho] = sum_j S[i][j][rho] Z[t][j][rho]
//
// The coupling reduces over the input blocks j, so a workgroup owns some rank indices of ALL blocks: a tile of 16 weight rows is
// 16 / JW rank indices of JW neighbouring blocks, 2, 4, 8 or 16 of them. The other operand is 16 / JW tokens of each of these blocks (one JW-th of
// the product is meant); with two blocks, up to 16 tokens of either (two MFMAs per step). The wavefronts take a tile of
// blocks each, or, with few tiles, a part of a tile's contraction index. Z goes through LDS once as [rho][t][j], where every rank index is one 16x16x16 MFMA against its 16x16
// coupling tile, and a lane then holds all 8 rank indices of four (token, output block): 16-byte stores.
//
// What bounds it: a launch, one memory latency and the fetch of instructions that run once, as in the kernel for the product
// alone (gemm_skinny.hip; the loops are rolled and operands come as direct loads for the same reason); what it saves is the
// coupling's launch.
#include "skinny_source.h"

namespace blr {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;

constexpr int FW_ZP = 40;                                // bytes per (rank index, token) of Z in LDS: 16 blocks, padded against bank conflicts

struct FewArgs {
    const bf16_t *X, *Vt, *Sp;
    bf16_t* A;
    int T, n_in, q, b, r;
    int pairs, pshift;                                   // tiles of JW input blocks ("pairs"); wavefront w takes part w >> pshift of pair w & ((1 << pshift) - 1)
    int splits, kper;                                    // parts of a pair's contraction index, indices per part (32 | kper)
    int slots;                                           // steps of 32 a wavefront's part of LDS holds
};

// JW: input blocks in a tile of 16 weight rows, 16 / JW rank indices each; XT: MFMAs per step, whose 16 XT columns are 16 XT / JW
// tokens of each of the blocks; SRC: where the tokens' rows come from (skinny_source.h; computed rows: XT = 1); TAIL: a wavefront's part of the contraction index is no whole number of steps; SPLIT: pairs are split
template <int XT, int SRC>
struct FewCfg {
    static constexpr int XL = SRC == kSrcInput ? XT : 0; // token rows that come as direct loads, per step
    static constexpr int SLOT = (1 + XL) * 1024;         // 16 weight rows and 16 XL token rows of 64 bytes
    static constexpr int SLOTS = XL == 2 ? 6 : 8;
};
template <int JW, int XT, int SRC, bool TAIL, bool SPLIT>
__global__ __launch_bounds__(512) void blast_few_kernel(FewArgs a, SkinnySource src) {
    using C = FewCfg<XT, SRC>;
    static_assert(SRC == kSrcInput || XT == 1, "computed rows: a handful of tokens");
    constexpr int XL = C::XL, SLOT = C::SLOT, SLOTS = C::SLOTS, RANKS = 16 / JW, TOK = 16 * XT / JW;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho0 = blockIdx.x * RANKS;
    const int split = SPLIT ? wave >> a.pshift : 0, pair = SPLIT ? wave & ((1 << a.pshift) - 1) : wave;
    const bool busy = pair < a.pairs && split < a.splits;                       // uniform
    const int j0 = JW * pair;
    auto block = [&](int i) { return j0 + i < a.b ? j0 + i : a.b - 1; };        // (an absent block repeats the last one; its Z is zero)
    const int kw = split * a.kper, kend = !busy ? 0 : a.q - kw < a.kper ? a.q - kw : a.kper;   // this wavefront's indices: [kw, kw + kend)
    const int steps = (kend + 31) >> 5;
    // A direct load fills 16 rows of 64 bytes: lane l brings the piece of slot l % 4 of row l / 4, pieces XOR-swizzled by the row
    const int lrow = lane >> 2, piece = (lane & 3) ^ ((lrow >> 2) & 3);
    const bf16_t* W = a.Vt + ((int64_t)block(lrow / RANKS) * a.r + rho0 + lrow % RANKS) * a.q + kw + piece * 8;
    const bf16_t* X[XL ? XL : 1];
#pragma unroll
    for (int x = 0; x < XL; ++x) {
        const int c = 16 * x + lrow, tok = c % TOK;
        X[x] = a.X + (int64_t)(tok < a.T ? tok : a.T - 1) * a.n_in + block(c / TOK) * a.q + kw + piece * 8;
    }
    unsigned char* mine = smem + wave * (a.slots * SLOT);
    int kf = 0;
    auto fetch = [&](unsigned char* slot) {
        // pieces past the part's end are zeros in both operands (an infinity times zero would be NaN)
        auto from = [&](const bf16_t* p) { return TAIL && kf + piece * 8 >= kend ? zero_piece : (const unsigned char*)(p + kf); };
        __builtin_amdgcn_global_load_lds(BLR_GPTR(from(W)), BLR_LPTR(slot), 16, 0, 0);
#pragma unroll
        for (int x = 0; x < XL; ++x) __builtin_amdgcn_global_load_lds(BLR_GPTR(from(X[x])), BLR_LPTR(slot + (1 + x) * 1024), 16, 0, 0);
        kf += 32;
    };
    const unsigned frag = (unsigned)(uintptr_t)BLR_LPTR(mine) + l16 * 64 + ((kg ^ ((l16 >> 2) & 3)) * 16);
    // computed rows [T][n_in] lie behind the wavefronts' slots
    const unsigned xs = a.n_in * 2 + 16;
    unsigned char* rows = smem + 8 * (a.slots * SLOT);
    const unsigned row_frag = (unsigned)(uintptr_t)BLR_LPTR(rows) + (l16 % TOK < a.T ? l16 % TOK : a.T - 1) * xs + (block(l16 / TOK) * a.q + kw) * 2;
    f32x4 acc[XT];
#pragma unroll
    for (int x = 0; x < XT; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](unsigned at, int t) {                // the step in the slot at `at`
        bf16x8 w = lds_read_frag(frag + at), xv[XT];
#pragma unroll
        for (int x = 0; x < XT; ++x) {
            if constexpr (XL > 0) xv[x] = lds_read_frag(frag + at + (1 + x) * 1024);
            else xv[x] = lds_read_frag(row_frag + (TAIL && t * 32 + kg * 8 >= kend ? 0 : t * 64 + kg * 16));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w) :: "memory");
#pragma unroll
        for (int x = 0; x < XT; ++x) asm volatile("" : "+v"(xv[x]));
        if (TAIL && XL == 0 && t * 32 + kg * 8 >= kend) xv[0] = bf16x8{};
#pragma unroll
        for (int x = 0; x < XT; ++x) acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, xv[x], acc[x], 0, 0, 0);
    };

    // the coupling's tiles: output block l16, input blocks 4 kg .. (older than the operands, so the waits below cover them)
    s16x4 sf[RANKS];
    if (wave == 0) {
        const bf16_t* S = a.Sp + (int64_t)rho0 * 256 + l16 * 16 + kg * 4;
#pragma unroll
        for (int e = 0; e < RANKS; ++e) sf[e] = *(const s16x4*)(S + e * 256);
    }
    int t = 0;
    for (; t < steps && t < a.slots; ++t) fetch(mine + t * SLOT);
    if constexpr (SRC != kSrcInput) {
        source_rows<SRC, 8>(src, a.T, a.n_in, 0, rows, xs, (float*)(rows + a.T * xs));
        __syncthreads();
    }
    t = 0;
    unsigned at = 0;
#pragma unroll 1
    for (; t + SLOTS < steps; ++t) {                     // (only with all SLOTS slots: what is in flight is a constant)
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"((1 + XL) * (SLOTS - 1)) : "memory");
        step(at, t);
        fetch(mine + at);
        at = at == (SLOTS - 1) * SLOT ? 0 : at + SLOT;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
    for (; t < steps; ++t) {
        step(at, t);
        at = at == (unsigned)(a.slots - 1) * SLOT ? 0 : at + SLOT;
    }
    __syncthreads();                                     // every wavefront is past its operands: Z and the partial sums take their place

    // accumulator element e of a lane: row 4 kg + e, i.e. rank index row % RANKS of the tile's block row / RANKS; column l16 of
    // product x: token c % TOK of block c / TOK, c = 16 x + l16
    unsigned char* Zs = smem;
    float* part = (float*)(smem + RANKS * 16 * FW_ZP); // [split][1 << pshift][row][16 + 1]
    auto put = [&](int rho, int tok, int j, float v) { *(bf16_t*)(Zs + (rho * 16 + tok) * FW_ZP + j * 2) = float_to_bf16(j < a.b ? v : 0.f); };
    if (a.pairs < 16 / JW)
#pragma unroll 1
        for (int it = tid; it < RANKS * 16 * 8; it += 512) {                    // blocks no pair has, two at a time
            const int j = it / (RANKS * 16) * 2;
            if (j >= JW * a.pairs) *(unsigned*)(Zs + it % (RANKS * 16) * FW_ZP + j * 2) = 0;
        }
    const f32x4 z = XT == 1 || kg < 2 ? acc[0] : acc[XT - 1];
    // column c of the tile's row: whose token of which block; the others are no product that is asked for
    auto keep = [&](int row, int col, int jt, float v) {
        const int rb = row / RANKS, c = col + (XT == 2 && row >= 8 ? 16 : 0);
        if (c / TOK == rb) put(row % RANKS, c % TOK, jt + rb, v);
    };
    if (SPLIT) {
#pragma unroll
        for (int e = 0; e < 4; ++e) part[(wave * 16 + 4 * kg + e) * 17 + l16] = z[e];
        __syncthreads();
#pragma unroll 1
        for (int it = tid; it < a.pairs * 256; it += 512) {      // (in the order of the parts: results do not depend on timing)
            const int row = (it >> 4) & 15, c = it & 15, at0 = (it >> 4) * 17 + c;
            float v = part[at0];
            for (int sp = 1; sp < a.splits; ++sp) v += part[((sp * 256) << a.pshift) / 16 * 17 + at0];
            keep(row, c, JW * (it >> 8), v);
        }
    } else if (busy) {
#pragma unroll
        for (int e = 0; e < 4; ++e) keep(4 * kg + e, l16, j0, z[e]);
    }
    __syncthreads();
    if (wave > 0) return;
    f32x4 d[RANKS];
#pragma unroll
    for (int e = 0; e < RANKS; ++e) {
        const s16x4 zf = *(const s16x4*)(Zs + (e * 16 + l16) * FW_ZP + kg * 8);
        d[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(sf[e], zf, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {                        // d[.][e]: token l16, output block 4 kg + e
        const int i = 4 * kg + e;
        if (l16 < a.T && i < a.b) {
            bf16_t* p = a.A + ((int64_t)l16 * a.b + i) * a.r + rho0;
            if constexpr (RANKS == 8) *(u32x4*)p = u32x4{pack2_bf16(d[0][e], d[1][e]), pack2_bf16(d[2][e], d[3][e]), pack2_bf16(d[4][e], d[5][e]), pack2_bf16(d[6][e], d[7][e])};
            else if constexpr (RANKS == 4) *(uint2*)p = make_uint2(pack2_bf16(d[0][e], d[1][e]), pack2_bf16(d[2][e], d[3][e]));
            else if constexpr (RANKS == 2) *(unsigned*)p = pack2_bf16(d[0][e], d[1][e]);
            else *p = float_to_bf16(d[0][e]);
        }
    }
}

template <int JW, int XT, int SRC, bool SPLIT>
hipError_t launch_few(FewArgs a, const SkinnySource& src, hipStream_t s) {
    using C = FewCfg<XT, SRC>;
    constexpr int RANKS = 16 / JW;
    const int steps = (a.kper + 31) / 32;
    a.slots = steps < C::SLOTS ? steps : C::SLOTS;
    int lds = 8 * a.slots * C::SLOT;
    if (SRC != kSrcInput) lds += a.T * (a.n_in * 2 + 16) + a.T * 8 * 4;
    const int sums = RANKS * 16 * FW_ZP + (SPLIT ? 8 * 16 * 17 * 4 : 0);
    if (lds < sums) lds = sums;
    static LdsLimitOnce lds_limit;
    if (hipError_t e = lds_limit.set({(const void*)blast_few_kernel<JW, XT, SRC, false, SPLIT>, (const void*)blast_few_kernel<JW, XT, SRC, true, SPLIT>}, 160 * 1024); e != hipSuccess) return e;
    const dim3 grid((unsigned)(a.r / RANKS));
    if (a.kper % 32 || a.q % a.kper) hipLaunchKernelGGL((blast_few_kernel<JW, XT, SRC, true, SPLIT>), grid, dim3(512), lds, s, a, src);
    else hipLaunchKernelGGL((blast_few_kernel<JW, XT, SRC, false, SPLIT>), grid, dim3(512), lds, s, a, src);
    return hipGetLastError();
}

FewArgs few_args(int jw, const void* X, const void* Vt, const void* Sp, void* A, int64_t T, int n_in, int b, int r) {
    FewArgs a{};
    a.X = (const bf16_t*)X; a.Vt = (const bf16_t*)Vt; a.Sp = (const bf16_t*)Sp; a.A = (bf16_t*)A;
    a.T = (int)T; a.n_in = n_in; a.q = n_in / b; a.b = b; a.r = r;
    a.pairs = (b + jw - 1) / jw;
    while ((1 << a.pshift) < a.pairs) ++a.pshift;
    const int most = 8 >> a.pshift, steps = (a.q + 31) / 32;
    a.kper = most > 1 ? 32 * ((steps + most - 1) / most) : a.q;
    a.splits = (a.q + a.kper - 1) / a.kper;             // (parts that have something to do)
    return a;
}

template <int JW, int XT, int SRC>
hipError_t launch_few(const FewArgs& a, const SkinnySource& src, hipStream_t s) {
    if constexpr (JW > 2) return launch_few<JW, XT, SRC, true>(a, src, s);   // (at most four tiles of blocks, and wide_tile's q: there are always parts)
    else return a.splits > 1 ? launch_few<JW, XT, SRC, true>(a, src, s) : launch_few<JW, XT, SRC, false>(a, src, s);
}

// How many blocks to a tile: more of them are more workgroups, r JW / 16, of fewer weights each, for fewer tokens. The most that the
// tokens leave and that stay one round, one workgroup to a compute unit (their LDS). Whole calls on graph replays with 2 / 4 / 8 / 16 blocks
// to a tile, 16 input blocks unless said: 1 token 8192 -> 768, r = 32 7.05 / 6.63 / 5.94 / 5.75 us, 8192 -> 2048, r = 384 7.44 / 6.98 / 6.37 /
// 6.43 (384 workgroups), 4096 x 4096, r = 256 6.23 / 6.16 / 5.87 / 5.78, r = 1024 6.92 / 6.94 / 6.87 / 7.63 (1024); 2 tokens 8192 -> 2048,
// r = 192 7.20 / 6.81 / 6.17; 4 tokens 3072 -> 768, 3 blocks, r = 128 6.62 / 6.15. With more than 8 blocks two to a tile need no sum of
// parts, and short ones are as fast that way: 4 tokens of 2048 x 2048, blocks of 128, r = 256 5.85 / 6.08, blocks of 256 level;
// 2 tokens, blocks of 128, r = 512 6.53 / 6.78 / 6.59.
bool wide_tile(int jw, int64_t T, int q, int b, int r) {
    return T * jw <= 16 && b > jw / 2 && (int64_t)r * jw <= 16 * 256 && q > 32 && (b <= 8 || q * jw >= 2048);
}

}  // namespace

hipError_t launch_blast_few(const void* X, const void* Vt, const void* Sp, void* A, int64_t T, int n_in, int b, int r, hipStream_t s) {
    if (T > kBlastFewTokens) return hipErrorInvalidValue;
    const int q = n_in / b;
    if (wide_tile(16, T, q, b, r)) return launch_few<16, 1, kSrcInput>(few_args(16, X, Vt, Sp, A, T, n_in, b, r), {}, s);
    if (wide_tile(8, T, q, b, r)) return launch_few<8, 1, kSrcInput>(few_args(8, X, Vt, Sp, A, T, n_in, b, r), {}, s);
    if (wide_tile(4, T, q, b, r)) return launch_few<4, 1, kSrcInput>(few_args(4, X, Vt, Sp, A, T, n_in, b, r), {}, s);
    const FewArgs a = few_args(2, X, Vt, Sp, A, T, n_in, b, r);
    return T <= 8 ? launch_few<2, 1, kSrcInput>(a, {}, s) : launch_few<2, 2, kSrcInput>(a, {}, s);
}

// (a row of T tokens and eight steps of eight wavefronts in LDS)
bool blast_few_norm_supported(int64_t T, int n_in) { return T >= 1 && T <= kSourceTokens && T * (n_in * 2 + 48) <= 96 * 1024; }

hipError_t launch_blast_few_norm(const SkinnySource& src, const void* Vt, const void* Sp, void* A, int64_t T, int n_in, int b, int r, hipStream_t s) {
    return launch_few<2, 1, kSrcNorm>(few_args(2, nullptr, Vt, Sp, A, T, n_in, b, r), src, s);
}

}  // namespace blr
