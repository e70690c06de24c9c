// The decoder-layer chain as one native object (include/blr_chain.h): the list of launches of a pass and their replay.
//
// What bounds a pass of few tokens is the number of launches: a launch costs 2.5 to 4 us of host time, and 1.6 us on the
// GPU inside a graph, as much as the work of one of these kernels. 16 BLAST layers at one token were 306 launches behind
// as many Python calls (1985 us a pass). The fused list needs 8 per layer, replayed as one graph.
#include "../../include/blr_chain.h"
#include "blr_common.h"
#include <cmath>
#include <exception>
#include <memory>
#include <mutex>
#include <vector>

using namespace blr;

struct blr_chain {
    blr_chain_desc d;
    std::vector<blr_chain_layer> layers;
    blr_chain_buffers buf;
    std::mutex lock;                                    // of the fields below
    int calls = 0;
    bool graph_failed = false;
    hipGraphExec_t exec = nullptr;
    hipEvent_t replayed = nullptr;                      // recorded behind every replay
};

namespace {

blr_status from_hip(hipError_t e) { return e == hipSuccess ? BLR_OK : BLR_ERR_LAUNCH; }

// A linear or group of the chain as its products
struct Linear {
    int n_in, n_out, r, members;
    bool in_blocked;                                    // Monarch: o and down
};
Linear linear_of(const blr_chain_desc& d, int which) {  // 0: q, k, v; 1: o; 2: gate, up; 3: down
    switch (which) {
        case 0: return {d.hidden, d.hidden, d.r_square, 3, false};
        case 1: return {d.hidden, d.hidden, d.r_square, 1, true};
        case 2: return {d.hidden, d.mlp, d.r_mlp, 2, false};
    }
    return {d.mlp, d.hidden, d.r_mlp, 1, true};
}

// ---- every step a call of the public entry points ----------------------------------------------------
blr_status run_linear(const blr_chain& c, const Linear& l, const blr_chain_factors& f, const void* X, void* Y, hipStream_t s) {
    const blr_chain_desc& d = c.d;
    void* ws = c.buf.workspace;
    const size_t wsb = c.buf.workspace_bytes;
    if (d.blast) {
        if (l.members > 1) return blr_blast_group_forward(X, f.second, f.first, Y, d.T, l.n_in, l.n_out, d.b, l.r, l.members, BLR_BF16, 0, ws, wsb, s);
        return blr_blast_forward(X, f.second, nullptr, f.first, Y, d.T, l.n_in, l.n_out, d.b, l.r, BLR_BF16, BLR_BLAST_PACKED, ws, wsb, s);
    }
    if (l.in_blocked) return blr_monarch_forward(X, f.first, f.second, Y, d.T, l.n_in, l.n_out, d.b, l.r, BLR_BF16, BLR_MONARCH_IN_BLOCKED, ws, wsb, s);
    return blr_monarch_rect_forward(X, f.first, f.second, Y, d.T, l.n_in, l.members * l.n_out, d.b, l.members * d.b, l.r / d.b, BLR_BF16,
                                    BLR_MONARCH_OUT_BLOCKED, ws, wsb, s);
}

blr_status run_steps(const blr_chain& c, hipStream_t s) {
    const blr_chain_desc& d = c.d;
    const blr_chain_buffers& b = c.buf;
    blr_status st = blr_rmsnorm(b.h, b.n, d.T, d.hidden, d.eps, BLR_BF16, s);
    const size_t col = (size_t)d.hidden * 2;
    for (int i = 0; i < d.layers && st == BLR_OK; ++i) {
        const blr_chain_layer& L = c.layers[i];
        auto step = [&](auto&& f) { if (st == BLR_OK) st = f(); };
        step([&] { return run_linear(c, linear_of(d, 0), L.qkv, b.n, b.qkv, s); });
        step([&] { return blr_sum3_scaled_ld(b.qkv, (char*)b.qkv + col, (char*)b.qkv + 2 * col, b.a, d.T, d.hidden, 3 * (int64_t)d.hidden, (float)(1.0 / std::sqrt(3.0)), BLR_BF16, s); });
        step([&] { return run_linear(c, linear_of(d, 1), L.o, b.a, b.o, s); });
        step([&] { return blr_residual_add_rmsnorm(b.h, b.o, b.n, d.T, d.hidden, d.eps, BLR_BF16, s); });
        step([&] { return run_linear(c, linear_of(d, 2), L.gate_up, b.n, b.gu, s); });
        step([&] { return blr_silu_mul_ld(b.gu, (char*)b.gu + (size_t)d.mlp * 2, b.m, d.T, d.mlp, 2 * (int64_t)d.mlp, BLR_BF16, s); });
        step([&] { return run_linear(c, linear_of(d, 3), L.down, b.m, b.dn, s); });
        step([&] { return blr_residual_add_rmsnorm(b.h, b.dn, i + 1 < d.layers ? b.n : nullptr, d.T, d.hidden, d.eps, BLR_BF16, s); });
    }
    return st;
}

// ---- a handful of tokens: two launches per linear, the step in front of a product inside it ----------
// stage 1 of a linear, its input to be computed by the source, and stage 2 (Monarch) or the coupling and stage 3 (BLAST)
struct Products { GemmDesc first, second; SkinnySource couple; };
Products products_of(const blr_chain& c, const Linear& l, const blr_chain_factors& f, void* Y) {
    const blr_chain_desc& d = c.d;
    const int b = d.b, p = l.n_in / b, q = l.n_out / b, T = (int)d.T, R = l.r * l.members;
    Products P{};
    GemmDesc &s1 = P.first, &s2 = P.second;
    s1.M = s2.M = T;
    s1.C = c.buf.workspace; s2.A = c.buf.workspace; s2.C = Y;
    if (d.blast) {
        const void *Vt, *Sc;
        blast_packed_parts(f.first, l.n_in, l.n_out, b, R, &Vt, &Sc);
        s1.B = Vt; s1.b_gs = (int64_t)p * R; s1.b_rs = p; s1.b_ks = 1;
        s1.c_rs = (int64_t)b * R; s1.c_gs = R; s1.c_div = 1; s1.c_hi = 1;
        s1.N = R; s1.K = p; s1.G = b;
        s2.B = f.second; s2.b_gs = (int64_t)q * l.r; s2.b_rs = l.r; s2.b_ks = 1;
        s2.c_rs = (int64_t)l.members * l.n_out; s2.c_gs = q; s2.c_div = 1; s2.c_hi = 1;
        s2.N = q; s2.K = l.r; s2.G = l.members * b;
        P.couple.a = (const bf16_t*)c.buf.workspace; P.couple.y = (const bf16_t*)Sc; P.couple.d = R; P.couple.b = b;
        return P;
    }
    const int b2 = l.members * b, rp = l.r / b;         // one Monarch layer with members * b output blocks
    s1.B = f.first; s1.b_gs = (int64_t)rp * b2 * p; s1.b_rs = p; s1.b_ks = 1; s1.b_div = rp; s1.b_mul = b2;
    s1.c_rs = (int64_t)b2 * l.r; s1.c_gs = rp; s1.c_div = rp; s1.c_hi = l.r; s1.c_lo = 1;
    s1.N = rp * b2; s1.K = p; s1.G = b;
    s2.a_gs = l.r; s2.a_rs = (int64_t)b2 * l.r;
    s2.B = f.second; s2.b_gs = (int64_t)q * l.r; s2.b_rs = l.r; s2.b_ks = 1;
    s2.c_rs = (int64_t)l.members * l.n_out; s2.c_div = 1;
    if (l.in_blocked) { s2.c_gs = 1; s2.c_hi = b; }     // o and down leave the canonical (interleaved) order
    else { s2.c_gs = q; s2.c_hi = 1; }
    s2.N = q; s2.K = l.r; s2.G = b2;
    return P;
}

// Up to this many tokens: every workgroup of a product repeats the step in front of it (the RMS norm reads 8 KB per token). A layer
// of the chains of 2048 / 8192, fused against step by step: BLAST 37.8 / 47.6 / 51.9 / 61.8 us against 44.7 / 58.1 / 58.6 / 59.3 at
// 1 / 4 / 5 / 8 tokens, Monarch 35.6 / 41.0 / 45.1 / 52.2 against 43.9 / 43.0 / 45.9 / 47.0 (behind from 6 tokens on).
constexpr int64_t kChainFusedTokens = 4;

bool fused_possible(const blr_chain& c) {
    const blr_chain_desc& d = c.d;
    if (d.T < 1 || d.T > kChainFusedTokens || d.hidden % 8 || d.mlp % 8) return false;
    for (int w = 0; w < 4; ++w) {
        const Linear l = linear_of(d, w);
        const blr_chain_factors& f = w == 0 ? c.layers[0].qkv : w == 1 ? c.layers[0].o : w == 2 ? c.layers[0].gate_up : c.layers[0].down;
        const Products P = products_of(c, l, f, c.buf.qkv);
        if (!skinny_source_supported(P.first) || !skinny_source_supported(P.second)) return false;
        if (!d.blast && l.in_blocked && (l.n_in / d.b / d.b) % 8) return false;               // 16-byte pieces inside a segment
        if (d.blast && (l.r * l.members) % 8) return false;
    }
    return true;
}

blr_status run_fused(const blr_chain& c, hipStream_t s) {
    const blr_chain_desc& d = c.d;
    const blr_chain_buffers& b = c.buf;
    blr_status st = BLR_OK;
    auto step = [&](hipError_t e) { if (e != hipSuccess) st = BLR_ERR_LAUNCH; };
    auto linear = [&](int which, const blr_chain_factors& f, int kind, const SkinnySource& src, void* Y) {
        const Products P = products_of(c, linear_of(d, which), f, Y);
        step(launch_gemm_skinny_from(kind, P.first, src, s));
        if (d.blast) step(launch_gemm_skinny_from(kSrcCoupling, P.second, P.couple, s));
        else step(launch_gemm_skinny(P.second, s));
    };
    // the residual stream moves between two buffers: a product's workgroups all read the old one, one of them writes the new one
    auto norm = [&](const void* h, const void* y, void* out) {
        SkinnySource n{};
        n.a = (const bf16_t*)h; n.y = (const bf16_t*)y; n.out = (bf16_t*)out; n.d = d.hidden; n.scale = d.eps;
        return n;
    };
    auto slices = [&](const void* t, int width, int members, float scale) {
        SkinnySource e{};
        e.a = (const bf16_t*)t; e.ld = (int64_t)members * width; e.slice = width; e.scale = scale;
        const int p = width / d.b;
        if (d.blast) { e.gs = p; e.seg = p; e.seg_stride = p; }                               // input block g: its own p elements
        else { e.gs = p / d.b; e.seg = p / d.b; e.seg_stride = p; }                           // blocked input: b runs of p/b elements
        return e;
    };
    for (int i = 0; i < d.layers && st == BLR_OK; ++i) {
        const blr_chain_layer& L = c.layers[i];
        if (i == 0) linear(0, L.qkv, kSrcNorm, norm(b.h, nullptr, nullptr), b.qkv);
        else linear(0, L.qkv, kSrcNorm, norm(b.h2, b.dn, b.h), b.qkv);
        linear(1, L.o, kSrcSum3, slices(b.qkv, d.hidden, 3, (float)(1.0 / std::sqrt(3.0))), b.o);
        linear(2, L.gate_up, kSrcNorm, norm(b.h, b.o, b.h2), b.gu);
        linear(3, L.down, kSrcSilu, slices(b.gu, d.mlp, 2, 1.f), b.dn);
    }
    if (st != BLR_OK) return st;
    return from_hip(launch_add(b.h2, b.dn, b.h, d.T * d.hidden, s));
}

blr_status run_pass(const blr_chain& c, hipStream_t s) { return fused_possible(c) ? run_fused(c, s) : run_steps(c, s); }

// The launches of a pass as a graph; null where the runtime refuses.
hipGraphExec_t capture(const blr_chain& c) {
    hipStream_t s = nullptr;
    hipGraph_t g = nullptr;
    hipGraphExec_t exec = nullptr;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return nullptr;
    if (hipStreamBeginCapture(s, hipStreamCaptureModeRelaxed) == hipSuccess) {
        const blr_status st = run_pass(c, s);
        if (hipStreamEndCapture(s, &g) == hipSuccess && st == BLR_OK && g) {
            if (hipGraphInstantiate(&exec, g, nullptr, nullptr, 0) != hipSuccess) exec = nullptr;
        }
        if (g) (void)hipGraphDestroy(g);
    }
    (void)hipStreamDestroy(s);
    (void)hipGetLastError();                            // a refusal is not the caller's error
    return exec;
}

}  // namespace

extern "C" {

blr_status blr_chain_create(const blr_chain_desc* desc, const blr_chain_layer* layers, const blr_chain_buffers* buffers, blr_chain** out) {
    if (!desc || !layers || !buffers || !out) return BLR_ERR_INVALID_ARG;
    const blr_chain_desc& d = *desc;
    if (d.layers <= 0 || d.T < 0 || d.hidden <= 0 || d.mlp <= 0 || d.b <= 0 || d.r_square <= 0 || d.r_mlp <= 0 || !(d.eps >= 0.f) ||
        d.hidden % d.b || d.mlp % d.b) return BLR_ERR_INVALID_ARG;
    const blr_chain_buffers& b = *buffers;
    for (const void* p : {b.h, b.h2, b.n, b.a, b.o, b.dn, b.qkv, b.gu, b.m, b.workspace})
        if (d.T > 0 && (!p || ((uintptr_t)p & 15))) return BLR_ERR_INVALID_ARG;
    for (int i = 0; i < d.layers; ++i)
        for (const blr_chain_factors& f : {layers[i].qkv, layers[i].o, layers[i].gate_up, layers[i].down})
            if (!f.first || !f.second || ((uintptr_t)f.first & 15) || ((uintptr_t)f.second & 15)) return BLR_ERR_INVALID_ARG;
    size_t need = 0;
    for (int w = 0; w < 4; ++w) {
        const Linear l = linear_of(d, w);
        size_t n;
        if (d.blast) {
            n = l.members > 1 ? blr_blast_group_workspace_bytes(d.T, l.n_in, l.n_out, d.b, l.r, l.members, BLR_BF16, 0)
                              : blr_blast_workspace_bytes(d.T, l.n_in, l.n_out, d.b, l.r, BLR_BF16, BLR_BLAST_PACKED);
            if (!n || !blr_blast_packed_bytes(l.n_in, l.n_out, d.b, l.r * l.members, BLR_BF16)) return BLR_ERR_UNSUPPORTED;
        } else {
            if (l.r % d.b || (l.n_in / d.b) % d.b) return BLR_ERR_UNSUPPORTED;
            n = l.members > 1 ? blr_monarch_rect_workspace_bytes(d.T, l.n_in, l.members * l.n_out, d.b, l.members * d.b, l.r / d.b, BLR_BF16)
                              : blr_monarch_workspace_bytes(d.T, l.n_in, l.n_out, d.b, l.r, BLR_BF16);
        }
        if (n > need) need = n;
    }
    if (b.workspace_bytes < need) return BLR_ERR_WORKSPACE;
    try {                                               // (no exception leaves a C entry)
        std::unique_ptr<blr_chain> c(new blr_chain);
        c->d = d;
        c->layers.assign(layers, layers + d.layers);
        c->buf = b;
        *out = c.release();
    } catch (const std::exception&) {
        return BLR_ERR_LAUNCH;
    }
    return BLR_OK;
}

blr_status blr_chain_forward(blr_chain* c, blr_stream stream) {
    if (!c) return BLR_ERR_INVALID_ARG;
    if (c->d.T == 0) return BLR_OK;
    hipStream_t s = (hipStream_t)stream;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cs) != hipSuccess) { (void)hipGetLastError(); cs = hipStreamCaptureStatusActive; }
    if (cs != hipStreamCaptureStatusNone) return run_pass(*c, s);
    hipGraphExec_t exec;
    {
        std::lock_guard<std::mutex> g(c->lock);
        // the first pass runs as separate launches: a chain that is used once pays for no graph
        if (c->calls++ >= 1 && !c->exec && !c->graph_failed) {
            c->exec = hipEventCreateWithFlags(&c->replayed, hipEventDisableTiming) == hipSuccess ? capture(*c) : nullptr;
            c->graph_failed = !c->exec;
            if (c->graph_failed && c->replayed) { (void)hipEventDestroy(c->replayed); c->replayed = nullptr; }
        }
        exec = c->exec;
    }
    if (!exec) return run_pass(*c, s);
    if (hipGraphLaunch(exec, s) != hipSuccess) return BLR_ERR_LAUNCH;
    return from_hip(hipEventRecord(c->replayed, s));
}

void blr_chain_destroy(blr_chain* c) {
    if (!c) return;
    if (c->exec) {
        // a replay may still be running; the wait is for it alone: one for the device breaks a capture under way on another stream
        (void)hipEventSynchronize(c->replayed);
        (void)hipEventDestroy(c->replayed);
        (void)hipGraphExecDestroy(c->exec);
    }
    delete c;
}

}  // extern "C"
