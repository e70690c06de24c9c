// The decoder-layer chain as one native object (include/blr_chain.h): the list of launches of a pass and their replay.
//
// What bounds a pass of few tokens is the number of launches: a launch costs 2.5 to 4 us of host time, and 1.6 us on the
// GPU inside a graph, as much as the work of one of these kernels. 16 BLAST layers at one token were 306 launches behind
// as many Python calls (1985 us a pass). The list below needs 8 per layer there, replayed as one graph.
#include "../../include/blr_chain.h"
#include "blr_common.h"
#include <cmath>
#include <exception>
#include <memory>
#include <mutex>
#include <vector>

using namespace blr;

namespace blr {
blr_status group_first(bool blast, const void* X, const void* first, const void* second, int64_t T, int n_in, int n_out, int b, int r, int members,
                       void* workspace, size_t workspace_bytes, hipStream_t s);
}

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
// gathered: X of a Monarch o or down lies block by block already
blr_status run_linear(const blr_chain& c, const Linear& l, const blr_chain_factors& f, const void* X, void* Y, hipStream_t s, bool gathered = false) {
    const blr_chain_desc& d = c.d;
    void* ws = c.buf.workspace;
    const size_t wsb = c.buf.workspace_bytes;
    if (d.blast) {
        if (l.members > 1) return blr_blast_group_forward(X, f.second, f.first, Y, d.T, l.n_in, l.n_out, d.b, l.r, l.members, BLR_BF16, 0, ws, wsb, s);
        return blr_blast_forward(X, f.second, nullptr, f.first, Y, d.T, l.n_in, l.n_out, d.b, l.r, BLR_BF16, BLR_BLAST_PACKED, ws, wsb, s);
    }
    if (l.in_blocked) return blr_monarch_forward(X, f.first, f.second, Y, d.T, l.n_in, l.n_out, d.b, l.r, BLR_BF16, gathered ? 0 : BLR_MONARCH_IN_BLOCKED, ws, wsb, s);
    return blr_monarch_rect_forward(X, f.first, f.second, Y, d.T, l.n_in, l.members * l.n_out, d.b, l.members * d.b, l.r / d.b, BLR_BF16,
                                    BLR_MONARCH_OUT_BLOCKED, ws, wsb, s);
}

// ---- up to a handful of tokens the RMS norm runs inside the product behind it ------------------------
// Every workgroup of that product repeats it (it reads 8 KB per token). A layer of the chains of 2048 / 8192, inside against as
// launches of its own: BLAST 39.1 us at 3 tokens, 41.0 against 39.4 at 4; Monarch 37.1 at 3, 39.1 against 37.8 at 4.
constexpr int64_t kChainNormTokens = 3;

// stage 1 of a Monarch group on the norm of the residual stream
GemmDesc monarch_first(const blr_chain& c, const Linear& l, const blr_chain_factors& f) {
    const int b = c.d.b, p = l.n_in / b, b2 = l.members * b, rp = l.r / b;   // one layer with members * b output blocks
    GemmDesc d{};
    d.M = c.d.T; d.N = rp * b2; d.K = p; d.G = b;
    d.B = f.first; d.b_gs = (int64_t)rp * b2 * p; d.b_rs = p; d.b_ks = 1; d.b_div = rp; d.b_mul = b2;
    d.C = c.buf.workspace; d.c_rs = (int64_t)b2 * l.r; d.c_gs = rp; d.c_div = rp; d.c_hi = l.r; d.c_lo = 1;
    return d;
}
bool norm_inside(const blr_chain& c, int which, const blr_chain_factors& f) {
    const blr_chain_desc& d = c.d;
    const Linear l = linear_of(d, which);
    if (d.T > kChainNormTokens || d.hidden % 8) return false;
    return d.blast ? blast_few_norm_supported(d.T, l.n_in) : skinny_source_supported(monarch_first(c, l, f));
}

// A group and the elementwise step behind it: 3 members, their scaled sum; 2, SiLU(first) * second. One launch for the last product
// and the step where the group runs that way (up to 32 tokens gemm_skinny_kernel, from 65 on the tiles), else a call each.
//
// gathered: an input block of a Monarch o or down is b runs of n_in / b^2 elements of the blocked order, and the matrix kernels read
// runs of whole steps of 32. Where they are none, the combined result leaves in the order in which the next linear's re-ordered
// factor counts, an input block in one piece. A layer of 768 / 3072 in 4 blocks (runs of 48) at 1 / 4 / 16 / 32 tokens 44.5 / 49.1 / 50.9 /
// 57.6 us with the runs (first products on the portable kernel), 25.6 / 29.1 / 30.2 / 33.3 in one piece; of 2048 / 8192 in 16 blocks (runs of 8)
// 47.6 / 54.4 / 58.8 / 70.6 and 34.2 / 38.6 / 43.1 / 52.3, at 1000 tokens 212 and 159.
struct Group { bool tail, gathered; GroupTail t; };
Group group_of(const blr_chain& c, int which, const blr_chain_factors& f, void* out) {
    const Linear l = linear_of(c.d, which);
    Group g{};
    g.tail = group_tail(c.d.blast, f.second, c.d.T, l.n_in, l.n_out, c.d.b, l.r, l.members, c.buf.workspace, c.buf.workspace_bytes, &g.t);
    GemmDesc& p = g.t.product;
    p.C = out;
    const int run = l.n_out / c.d.b / c.d.b;
    if (!c.d.blast && run % 32) {
        p.c_gs = p.c_div = run; p.c_hi = l.n_out / c.d.b; p.c_lo = 1;
        g.gathered = true;
    }
    g.tail = g.tail && gemm_combine_supported(p, l.members);
    g.gathered = g.gathered && g.tail;
    return g;
}
blr_status run_group(const blr_chain& c, int which, const blr_chain_factors& f, const SkinnySource* norm, void* wide, void* out, hipStream_t s) {
    const blr_chain_desc& d = c.d;
    const Linear l = linear_of(d, which);
    const Group g = group_of(c, which, f, out);
    const float scale = l.members == 3 ? (float)(1.0 / std::sqrt(3.0)) : 1.f;
    blr_status st;
    if (!g.tail) {
        st = run_linear(c, l, f, c.buf.n, wide, s);
        if (st != BLR_OK) return st;
        char* w = (char*)wide;
        const size_t col = (size_t)l.n_out * 2;
        if (l.members == 3) return blr_sum3_scaled_ld(w, w + col, w + 2 * col, out, d.T, l.n_out, 3 * (int64_t)l.n_out, scale, BLR_BF16, s);
        return blr_silu_mul_ld(w, w + col, out, d.T, l.n_out, 2 * (int64_t)l.n_out, BLR_BF16, s);
    }
    if (norm && d.blast) {
        const void *Vt, *Sp;
        blast_packed_parts(f.first, l.n_in, l.n_out, d.b, l.r * l.members, &Vt, &Sp);
        st = from_hip(launch_blast_few_norm(*norm, Vt, Sp, (void*)g.t.product.A, d.T, l.n_in, d.b, l.r * l.members, s));
    } else if (norm) {
        st = from_hip(launch_gemm_skinny_norm(monarch_first(c, l, f), *norm, s));
    } else {
        st = group_first(d.blast, c.buf.n, f.first, f.second, d.T, l.n_in, l.n_out, d.b, l.r, l.members, c.buf.workspace, c.buf.workspace_bytes, s);
    }
    return st != BLR_OK ? st : from_hip(launch_gemm_combine(g.t.product, l.members, {g.t.a_ms, g.t.b_ms, scale}, s));
}

blr_status run_pass(const blr_chain& c, hipStream_t s) {
    const blr_chain_desc& d = c.d;
    const blr_chain_buffers& b = c.buf;
    const blr_chain_layer& L0 = c.layers[0];
    const Group qkv = group_of(c, 0, L0.qkv, b.a), gate_up = group_of(c, 2, L0.gate_up, b.m);     // (every layer's: the same sizes, and all factors are aligned)
    const bool inside = qkv.tail && gate_up.tail && norm_inside(c, 0, L0.qkv) && norm_inside(c, 2, L0.gate_up);
    blr_status st = BLR_OK;
    auto step = [&](auto&& f) { if (st == BLR_OK) st = f(); };
    // inside: the residual stream moves between two buffers, the workgroups of a product all read the old one, one of them writes the new one
    auto norm = [&](const void* h, const void* y, void* out) {
        SkinnySource n{};
        n.a = (const bf16_t*)h; n.y = (const bf16_t*)y; n.out = (bf16_t*)out; n.d = d.hidden; n.scale = d.eps;
        return n;
    };
    if (!inside) st = blr_rmsnorm(b.h, b.n, d.T, d.hidden, d.eps, BLR_BF16, s);
    for (int i = 0; i < d.layers && st == BLR_OK; ++i) {
        const blr_chain_layer& L = c.layers[i];
        const bool last = i + 1 == d.layers;
        const SkinnySource n1 = i ? norm(b.h2, b.dn, b.h) : norm(b.h, nullptr, nullptr), n2 = norm(b.h, b.o, b.h2);
        step([&] { return run_group(c, 0, L.qkv, inside ? &n1 : nullptr, b.qkv, b.a, s); });
        step([&] { return run_linear(c, linear_of(d, 1), L.o, b.a, b.o, s, qkv.gathered); });
        if (!inside) step([&] { return blr_residual_add_rmsnorm(b.h, b.o, b.n, d.T, d.hidden, d.eps, BLR_BF16, s); });
        step([&] { return run_group(c, 2, L.gate_up, inside ? &n2 : nullptr, b.gu, b.m, s); });
        step([&] { return run_linear(c, linear_of(d, 3), L.down, b.m, b.dn, s, gate_up.gathered); });
        if (!inside) step([&] { return blr_residual_add_rmsnorm(b.h, b.dn, last ? nullptr : b.n, d.T, d.hidden, d.eps, BLR_BF16, s); });
    }
    if (inside) step([&] { return from_hip(launch_add(b.h2, b.dn, b.h, d.T * d.hidden, s)); });
    return st;
}

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
            n = blast_workspace_least(d.T, l.n_in, l.n_out, d.b, l.r * l.members);
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
