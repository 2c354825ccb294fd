// C ABI of the ZeCO hot path (declared in include/zeco.h): argument validation and dispatch to
// the gfx950 kernels.  Validation happens before any HIP call so that the error paths can be
// exercised on a host without a GPU.
#include "../../include/zeco.h"
#include "zeco_internal.h"

#include <atomic>

// Scratch of zeco_state_scan_tree_static, the entry point for callers that cannot allocate: a fixed array in
// the library's device image, one copy per GPU the library runs on, held until the process ends.  In host
// code this name only identifies the symbol - it is not a device address; the address on the current GPU
// comes from hipGetSymbolAddress (static_scratch() below) and that pointer is what the launches are given.
constexpr size_t kStaticScratchBytes = (size_t)33 << 20;
static __device__ __align__(256) unsigned char zeco_static_scratch[kStaticScratchBytes];

namespace {

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool dim_ok(int d) { return d == 64 || d == 128; }

// ZECO_OK when the descriptor is well formed and supported.  `any_length`: the entry point takes segment
// lengths that are no multiple of the chunk size (the forward entry points do, from 64 tokens on).
zeco_status check_desc(const zeco_gla_desc *d, bool any_length = false) {
    if (!d) return ZECO_ERR_INVALID_ARG;
    if (d->B < 0 || d->P <= 0 || d->H <= 0 || d->L <= 0 || d->d_k <= 0 || d->d_v <= 0 || d->C <= 0)
        return ZECO_ERR_INVALID_ARG;   // (B = 0, an empty batch, is valid: every entry point returns at once)
    if (d->io_dtype != ZECO_F32 && d->io_dtype != ZECO_BF16) return ZECO_ERR_INVALID_ARG;
    if (d->g_dtype != ZECO_F32 && d->g_dtype != ZECO_BF16) return ZECO_ERR_INVALID_ARG;
    if (!(d->scale == d->scale)) return ZECO_ERR_INVALID_ARG;
    if ((int64_t)d->P * d->L > (int64_t)1 << 40 || d->L > (1 << 30)) return ZECO_ERR_INVALID_ARG;
    const int64_t s[6] = {d->stride_b, d->stride_t, d->stride_h, d->vstride_b, d->vstride_t, d->vstride_h};
    for (int i = 0; i < 6; ++i)
        if (s[i] < 0 || s[i] % 8 != 0) return ZECO_ERR_INVALID_ARG;
    if (d->stride_h < d->d_k || d->vstride_h < d->d_v) return ZECO_ERR_INVALID_ARG;
    if (d->stride_t < d->d_k || d->vstride_t < d->d_v) return ZECO_ERR_INVALID_ARG;
    // the kernels keep in-chunk offsets (64 tokens x stride_t elements) in 32 bits
    if (d->stride_t > ((int64_t)1 << 24) || d->vstride_t > ((int64_t)1 << 24)) return ZECO_ERR_UNSUPPORTED;
    if ((int64_t)d->B * d->P * d->H > (int64_t)1 << 24) return ZECO_ERR_INVALID_ARG;
    // chunk length: 64 for bf16 (one token per lane of a wavefront); the fp32 kernel also takes 16 and 32
    const bool chunk_ok = d->C == 64 || (d->io_dtype == ZECO_F32 && (d->C == 16 || d->C == 32));
    if (!chunk_ok || !dim_ok(d->d_k) || !dim_ok(d->d_v)) return ZECO_ERR_UNSUPPORTED;
    if (d->L % d->C != 0 && !any_length) return ZECO_ERR_UNSUPPORTED;
    if (d->L < 64) return ZECO_ERR_UNSUPPORTED;   // (the correction works on windows of 64 tokens inside a segment)
    if (d->io_dtype == ZECO_F32 && d->g_dtype != ZECO_F32) return ZECO_ERR_UNSUPPORTED;
    if (d->g_per_head != 0 && d->g_per_head != 1) return ZECO_ERR_INVALID_ARG;
    if (d->g_per_head && (d->io_dtype != ZECO_BF16 || d->g_dtype != ZECO_F32)) return ZECO_ERR_UNSUPPORTED;
    if (d->wide_gates != 0 && d->wide_gates != 1) return ZECO_ERR_INVALID_ARG;
    return ZECO_OK;
}

int gate_mode(const zeco_gla_desc *d) {
    if (d->g_per_head) return zeco::kGateHead;
    return d->g_dtype == ZECO_BF16 ? zeco::kGateBF16 : zeco::kGateF32;
}

// the same with the descriptor's choice of range, for the bf16 chunk kernel
int chunk_gate(const zeco_gla_desc *d) { return gate_mode(d) | (d->wide_gates ? zeco::kGateWide : 0); }

zeco_status from_hip(hipError_t e) { return e == hipSuccess ? ZECO_OK : ZECO_ERR_HIP; }

int chunks_of(int L) { return (L + 63) / 64; }

// Segment length of a chunk-kernel launch: chunks, and how far the first one falls short of 64 tokens.
void set_length(zeco::ChunkParams &p, int L) {
    p.L = L; p.n_chunks = chunks_of(L); p.pad = 64 * p.n_chunks - L;
}
// The same in chunks of C tokens (the fp32 kernel).
void set_length_c(zeco::ChunkParams &p, int L, int C) {
    p.L = L; p.n_chunks = (L + C - 1) / C; p.pad = C * p.n_chunks - L;
}

int gate_mode(const zeco_gla_desc *d);
int chunk_gate(const zeco_gla_desc *d);
// One of the phases both precisions have (0 local pass, 1 states only, 2 output pass from S_init, 3 backward
// state pass; fp32 only: 4 dV pass), on the segments p describes (p.L tokens each, or the table p.seg_start).
hipError_t launch_phase(zeco::ChunkParams &p, const zeco_gla_desc *d, int mode, hipStream_t s) {
    if (d->io_dtype == ZECO_F32) {
        if (!p.cut.n) set_length_c(p, p.L, zeco::f32_chunk(p, d->C, mode));
        return zeco::launch_chunk_f32(p, d->d_k, d->d_v, d->C, mode, s);
    }
    return zeco::launch_chunk_bf16(p, d->d_k, d->d_v, chunk_gate(d), mode, s);
}

// Segments per group of the two-level scan: the divisor g of P that minimises the length of the serial
// work, 2 g + P / g (two passes inside the groups, one over the groups).  Returns P when no proper divisor helps.
int tree_group(int P) {
    int best = P;
    long long cost = P;                       // the plain chain
    auto consider = [&](int g) {
        const long long c = 2ll * g + P / g;
        if (c < cost || (c == cost && g < best)) { cost = c; best = g; }
    };
    for (int a = 2; (long long)a * a <= P; ++a) {   // divisor pairs (a, P / a)
        if (P % a) continue;
        consider(a);
        consider(P / a);
    }
    return best;
}

// Floats of scratch the two-level scan of a chain of P segments needs (0: the chain is not split).
size_t tree_floats(int P, int BH, int d_k, int d_v, int gate_per_head) {
    const int g = tree_group(P);
    if (g == P) return 0;
    const size_t J = P / g, state = (size_t)BH * d_k * d_v;
    return 2 * J * state + J * (size_t)BH * (gate_per_head ? 1 : d_k);
}

// The two-level scan of one chain (sp.groups == 1, sp.P segments): every group of g segments from the zero
// state (end state and total log decay), the chain over the groups, every group again from the state
// entering it.  `scratch`: tree_floats() floats.
hipError_t launch_scan_tree(zeco::ScanParams sp, float *scratch, hipStream_t s) {
    const int P = sp.P, g = tree_group(P), J = P / g;
    const size_t state = (size_t)sp.BH * sp.d_k * sp.d_v;
    float *T = scratch, *I = T + J * state, *Gt = I + J * state;
    zeco::ScanParams p = sp;
    p.G_pre = nullptr;
    p.S0 = nullptr; p.S_init = nullptr; p.S_last = T; p.S_last2 = nullptr; p.G_sum = Gt; p.P = g; p.groups = J;
    hipError_t e = zeco::launch_scan(p, s);
    if (e != hipSuccess) return e;
    p.S_loc = T; p.G_tot = Gt; p.S0 = sp.S0; p.S_init = I; p.S_last = sp.S_last; p.S_last2 = sp.S_last2; p.G_sum = nullptr;
    p.P = J; p.groups = 1;
    if ((e = zeco::launch_scan(p, s)) != hipSuccess) return e;
    p.S_loc = sp.S_loc; p.G_tot = sp.G_tot; p.S0 = I; p.S_init = sp.S_init; p.S_last = p.S_last2 = nullptr;
    p.P = g; p.groups = J;
    return zeco::launch_scan(p, s);
}

// Inside the fused calls: is the chain of P pieces better scanned as a tree?  Only for a single head of up to 8192
// elements, whose chain, though split over the waves of a workgroup, is bound by the latency of its steps: scan / tree, us, 256,
// 512, 1024, 4096 segments of 64 x 64 9.8 / 13.2, 17.5 / 15.9, 34 / 19, 135 / 52; of 128 x 64 10.4 / 13.9, 19.4 / 19.0, 38 / 28, 138 / 82; of
// 128 x 128 12.1 / 17.6, 22.5 / 25.2, 41 / 46, 149 / 159.
bool chain_wants_tree(int P, int BH, int d_k, int d_v) {
    if (!(BH == 1 && P >= 512 && d_k * d_v <= 8192)) return false;
    const int g = tree_group(P);
    return g != P && P / g <= 65535;          // (the groups are the y dimension of the launch)
}
size_t chain_scratch_floats(int P, int BH, int d_k, int d_v, int gate_per_head) {
    return chain_wants_tree(P, BH, d_k, d_v) ? tree_floats(P, BH, d_k, d_v, gate_per_head) : 0;
}
hipError_t launch_scan_chain(const zeco::ScanParams &sp, float *scratch, hipStream_t s) {
    return chain_wants_tree(sp.P, sp.BH, sp.d_k, sp.d_v) ? launch_scan_tree(sp, scratch, s) : zeco::launch_scan(sp, s);
}

// Device address of zeco_static_scratch on the current GPU.  Every GPU has its own copy of the array at its
// own address, so the address is looked up once per device, with that device current, and kept.  (Two
// threads that make a device's first call together both look up the same address; no lock is needed.)
constexpr int kMaxDevices = 64;
std::atomic<void *> g_static_scratch[kMaxDevices];
hipError_t static_scratch(void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void *ptr = g_static_scratch[dev].load(std::memory_order_acquire);
    if (!ptr) {
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(zeco_static_scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_static_scratch[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return hipSuccess;
}

}  // namespace

extern "C" {

constexpr long long kComputeUnits = 256;

static int subsegments(const zeco_gla_desc *d);
static zeco::Cut cut_of(long long tokens, long long n);
static void set_cut(zeco::ChunkParams &p, const zeco::Cut &c);
static int longest_tokens(const zeco::Cut &c);
static size_t bwd_checkpoint_floats(const zeco_gla_desc *d, int P, int L);

// With one decay per head and between 65 and 128 streams the local pass runs every segment as two halves
// from the zero state on whole workgroups (256 streams), then corrects the second halves' outputs with the
// first halves' end states where their decay has not vanished, and rebases the second halves' G_cum, which
// costs 4 bytes per token and head in this layout: sibling workgroups on 128 streams leave the kernel bound
// by its own pipeline (3.3 TB/s at c3), whole workgroups on 256 streams move 5.4 TB/s.
static bool halves_with_correction(const zeco_gla_desc *d) {
    if (d->io_dtype != ZECO_BF16 || !d->g_per_head || d->d_v != 128) return false;
    const long long streams = (long long)d->B * d->P * d->H;
    return streams > 64 && streams <= 128 && d->L % 128 == 0 && d->L / 2 >= 4096;
}

struct SubLayout {          // workspace carve-up, in floats
    size_t states, gates;   // elements of one state array / one gate array over all sub-segments
    size_t off_Ssub, off_Sinit, off_Gtot, off_Gpre, total;
};
static SubLayout sub_layout(const zeco_gla_desc *d, int S) {
    SubLayout w;
    const size_t n = (size_t)d->P * S * d->B * d->H;
    w.states = n * d->d_k * d->d_v;
    w.gates = 2 * n * d->d_k;   // (pairs)
    w.off_Ssub = 0;
    w.off_Sinit = w.off_Ssub + w.states;
    w.off_Gtot = w.off_Sinit + w.states;
    w.off_Gpre = w.off_Gtot + w.gates;
    w.total = w.off_Gpre + w.gates;
    return w;
}

static void fill_apply_params(zeco::ApplyParams &p, const zeco_gla_desc *d, int P, int L);

size_t zeco_gla_local_fwd_workspace(const zeco_gla_desc *desc) {
    if (check_desc(desc, true) != ZECO_OK) return 0;
    if (halves_with_correction(desc)) return sub_layout(desc, 2).total * sizeof(float);
    const int S = subsegments(desc);
    return S > 1 ? sub_layout(desc, S).total * sizeof(float) : 0;
}

zeco_status zeco_gla_local_fwd(const zeco_gla_desc *d, const void *q, const void *k, const void *v,
                               const void *g, void *o, float *S_loc, float *G_cum, float *G_tot,
                               void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !o || !S_loc || !G_cum || !G_tot) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(o) ||
        !aligned16(S_loc) || !aligned16(G_cum) || !aligned16(G_tot))
        return ZECO_ERR_INVALID_ARG;
    const size_t need = zeco_gla_local_fwd_workspace(d);
    int S = subsegments(d);
    if (workspace_bytes < need || (need && (!workspace || !aligned16(workspace)))) {
        // fp32, and lengths that do not halve, can do without: one chain a stream
        const bool must = halves_with_correction(d) || (d->io_dtype == ZECO_BF16 && d->L % (d->L % 64 ? 2 : 128) == 0);
        if (must) return workspace_bytes < need ? ZECO_ERR_WORKSPACE : ZECO_ERR_INVALID_ARG;
        S = 1;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);

    zeco::ChunkParams p;
    p.q = q; p.k = k; p.v = v; p.g = g; p.o = o;
    p.S_loc = S_loc; p.G_cum = G_cum; p.G_tot = G_tot; p.S_init = nullptr;
    p.B = d->B; p.P = d->P; p.H = d->H; p.T = (long long)d->P * d->L;
    set_length(p, d->L);
    p.scale = d->scale; p.kscale = 1.f;
    p.sb = d->stride_b; p.st = d->stride_t; p.sh = d->stride_h;
    p.vb = d->vstride_b; p.vt = d->vstride_t; p.vh = d->vstride_h;
    if (S == 1 && d->io_dtype == ZECO_F32) return from_hip(launch_phase(p, d, 0, s));
    if (halves_with_correction(d)) {
        const SubLayout w = sub_layout(d, 2);
        float *ws = static_cast<float *>(workspace);
        float *Ssub = ws + w.off_Ssub, *Sinit = ws + w.off_Sinit, *Gtot = ws + w.off_Gtot, *Gpre = ws + w.off_Gpre;
        // the halves from the zero state: o, G_cum counted from each half's first token, end states
        p.P = d->P * 2; set_length(p, d->L / 2);
        p.S_loc = Ssub; p.G_tot = Gtot;
        if (zeco::launch_chunk_bf16(p, d->d_k, d->d_v, chunk_gate(d), 0, s) != hipSuccess) return ZECO_ERR_HIP;
        // chain of the two halves of every segment: the state and the log decay entering the second half,
        // the segment's end state and total
        zeco::ScanParams sp;
        sp.S_loc = Ssub; sp.G_tot = Gtot; sp.S0 = nullptr; sp.S_init = Sinit; sp.S_last = S_loc;
        sp.P = 2; sp.groups = d->P; sp.BH = d->B * d->H; sp.d_k = d->d_k; sp.d_v = d->d_v;
        sp.rows_per_block = d->d_k / 16; sp.gate_per_head = 1;
        sp.G_pre = Gpre; sp.G_sum = G_tot;
        if (zeco::launch_scan(sp, s) != hipSuccess) return ZECO_ERR_HIP;
        // second halves (every other piece): o += (scale q .* exp(G_cum)) S_entering, with G_cum still counted
        // from the half's first token
        zeco::ApplyParams ap;
        fill_apply_params(ap, d, d->P * 2, d->L / 2);
        ap.q = q; ap.G_cum = G_cum; ap.S_init = Sinit; ap.o = o; ap.p0 = 1; ap.seg_step = 2;
        if (zeco::launch_apply_bf16(ap, d->d_k, d->d_v, s) != hipSuccess) return ZECO_ERR_HIP;
        return from_hip(zeco::launch_gate_offset_head(G_cum, Gpre, d->B, (long long)d->P * d->L, d->H, d->L / 2, s));
    }
    if (S == 1) return from_hip(zeco::launch_chunk_bf16(p, d->d_k, d->d_v, chunk_gate(d), 0, s));

    // Few streams: P*S sub-segments of L/S tokens, Alg. 1's schedule applied inside each segment: the
    // sub-segments' end states and total decays from the zero state, their scan inside the segment,
    // then the output pass of every sub-segment from its scanned state, which also writes G_cum counted
    // from the segment's first token.
    const SubLayout w = sub_layout(d, S);
    float *ws = static_cast<float *>(workspace);
    float *Ssub = ws + w.off_Ssub, *Sinit = ws + w.off_Sinit, *Gtot = ws + w.off_Gtot, *Gpre = ws + w.off_Gpre;
    set_cut(p, cut_of(d->L, S));
    p.P = d->P * S;
    p.S_loc = Ssub; p.G_tot = Gtot; p.pairs = 1; p.local = 1;
    hipError_t e = launch_phase(p, d, 1, s);
    if (e != hipSuccess) return ZECO_ERR_HIP;

    zeco::ScanParams sp;   // one chain of S sub-segments per segment; its end state is the segment's S_loc
    sp.S_loc = Ssub; sp.G_tot = Gtot; sp.S0 = nullptr; sp.S_init = Sinit; sp.S_last = S_loc;
    sp.P = S; sp.groups = d->P; sp.BH = d->B * d->H; sp.d_k = d->d_k; sp.d_v = d->d_v;
    sp.rows_per_block = d->d_k / 16; sp.gate_per_head = d->g_per_head;
    sp.G_pre = Gpre; sp.G_sum = G_tot;   // log decay preceding each sub-segment; the segment's total
    sp.pairs = 1;
    if ((e = zeco::launch_scan(sp, s)) != hipSuccess) return ZECO_ERR_HIP;

    p.S_loc = nullptr; p.G_tot = nullptr; p.S_init = Sinit;
    p.G_off = Gpre;
    return from_hip(launch_phase(p, d, 5, s));
}

// ---- two-phase forward ------------------------------------------------------------------------------
static void fill_chunk_params(zeco::ChunkParams &p, const zeco_gla_desc *d) {
    p.q = p.k = p.v = p.g = nullptr; p.o = nullptr;
    p.S_loc = p.G_cum = p.G_tot = nullptr; p.S_init = nullptr;
    p.B = d->B; p.P = d->P; p.H = d->H; p.T = (long long)d->P * d->L;
    set_length(p, d->L);
    p.scale = d->scale; p.kscale = 1.f;
    p.sb = d->stride_b; p.st = d->stride_t; p.sh = d->stride_h;
    p.vb = d->vstride_b; p.vt = d->vstride_t; p.vh = d->vstride_h;
}

// Tokens per workgroup of the correction: the largest of cap..64 (powers of two) that divides L, or, when the
// segments need not divide evenly (a ragged L, unequal segments), that is not above L - the last workgroup
// of a segment then has fewer blocks.  1024 where the call stops at the vanished decay (fewer workgroups
// that find nothing to do), 256 where it streams every token (measured 4 % faster there).
static void set_apply_share(zeco::ApplyParams &p, int L, int cap, bool divide) {
    int tpw = cap;
    if (divide) {
        while (tpw > 64 && L % tpw != 0) tpw >>= 1;
    } else {
        while (tpw > 64 && tpw > L) tpw >>= 1;
    }
    p.tokens_per_wg = tpw;
    p.wgs_per_seg = (64 * p.n_chunks + tpw - 1) / tpw;
}

// Correction over P segments of L tokens each (the caller's, or the pieces of a fused call).
static void fill_apply_params(zeco::ApplyParams &p, const zeco_gla_desc *d, int P, int L) {
    p.B = d->B; p.P = P; p.H = d->H; p.L = L; p.T = (long long)d->P * d->L;
    p.p0 = 0; p.gate_per_head = d->g_per_head; p.dense = 0;
    p.n_chunks = chunks_of(L); p.pad = 64 * p.n_chunks - L;
    set_apply_share(p, L, 1024, p.pad == 0);
    p.scale = d->scale;
    p.sb = d->stride_b; p.st = d->stride_t; p.sh = d->stride_h;
    p.vb = d->vstride_b; p.vt = d->vstride_t; p.vh = d->vstride_h;
}

// The building blocks over few streams: a stream is a serial chain of chunks, so with fewer of them than compute units most
// of the chip idles (64 streams of 8192 tokens, d = 128: states 172, output pass 324, gradients 1200 us).  With a workspace each
// call treats every segment as the one-call forms treat the whole run: it is cut into S pieces (block_pieces), the states
// entering the pieces come from their own end states and a scan inside the segment (one chain per segment), and the pass then
// runs over the pieces.  What the caller sees - one state per segment - stays what it is.
static int block_pieces(const zeco_gla_desc *d, int call);

struct BlockLayout {   // workspace carve-up, in floats
    int S;             // pieces per segment (1: the call is not cut and needs none of this)
    size_t state, off_Sinit, off_dSin, off_Gtot, off_ck, total;
};
static BlockLayout block_layout(const zeco_gla_desc *d, int call) {
    BlockLayout w;
    w.S = block_pieces(d, call);
    const size_t n = (size_t)d->P * w.S * d->B * d->H;
    w.state = (size_t)d->d_k * d->d_v;
    const bool states = call == ZECO_BLOCK_FWD_FROM_STATE || call == ZECO_BLOCK_BWD_FROM_STATE;
    w.off_Sinit = n * w.state;                                        // end states (later state gradients) of the pieces first
    w.off_dSin = w.off_Sinit + (states ? n * w.state : 0);
    w.off_Gtot = w.off_dSin + (call == ZECO_BLOCK_BWD_FROM_STATE ? n * w.state : 0);
    w.off_ck = w.off_Gtot + 2 * n * d->d_k;                           // (pairs)
    w.total = w.off_ck;
    if (call == ZECO_BLOCK_BWD_FROM_STATE)
        w.total += bwd_checkpoint_floats(d, d->P * w.S, longest_tokens(cut_of(d->L, w.S)));
    if (call == ZECO_BLOCK_BWD_FROM_STATE && w.total < bwd_checkpoint_floats(d, d->P, d->L)) w.total = bwd_checkpoint_floats(d, d->P, d->L);
    return w;
}

size_t zeco_gla_block_workspace(const zeco_gla_desc *desc, int32_t call) {
    if (check_desc(desc, true) != ZECO_OK || desc->B == 0 || call < 0 || call > ZECO_BLOCK_BWD_FROM_STATE) return 0;
    const BlockLayout w = block_layout(desc, call);
    if (w.S > 1) return w.total * sizeof(float);
    return call == ZECO_BLOCK_BWD_FROM_STATE ? zeco_gla_bwd_from_state_workspace(desc) : 0;
}

// Is the workspace one that the call can cut with?  (A smaller one, or none, is no error: the segments are then run whole.)
static bool block_cut(BlockLayout &w, const zeco_gla_desc *d, int call, const void *workspace, size_t bytes) {
    if (!workspace || !aligned16(workspace)) return false;
    w = block_layout(d, call);
    return w.S > 1 && bytes >= w.total * sizeof(float);
}

// The scan of the pieces of every segment: P chains of S.
static void fill_block_scan(zeco::ScanParams &sp, const zeco_gla_desc *d, int S) {
    sp.P = S; sp.groups = d->P; sp.BH = d->B * d->H; sp.d_k = d->d_k; sp.d_v = d->d_v;
    sp.rows_per_block = d->d_k / 16; sp.gate_per_head = d->g_per_head;
    sp.S0 = nullptr; sp.S_init = sp.S_last = nullptr;
}

// States entering the pieces of all segments (w.off_Sinit), from the states entering the segments.
static hipError_t block_entering_states(zeco::ChunkParams &p, const BlockLayout &w, float *ws, const zeco_gla_desc *d,
                                        const void *k, const void *v, const void *g, const float *S_init, hipStream_t s) {
    p.k = k; p.v = v; p.g = g; p.S_loc = ws; p.G_tot = ws + w.off_Gtot;
    p.skip_last = w.S;   // (what leaves a segment's last piece enters none of its pieces)
    hipError_t e = launch_phase(p, d, 1, s);
    if (e != hipSuccess) return e;
    p.skip_last = 0;
    zeco::ScanParams sp;
    fill_block_scan(sp, d, w.S);
    sp.S_loc = ws; sp.G_tot = ws + w.off_Gtot; sp.S0 = S_init; sp.S_init = ws + w.off_Sinit;
    return zeco::launch_scan(sp, s);
}

zeco_status zeco_gla_local_state_ws(const zeco_gla_desc *d, const void *k, const void *v, const void *g,
                                    float *S_loc, float *G_tot, void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!k || !v || !g || !S_loc || !G_tot) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(S_loc) || !aligned16(G_tot))
        return ZECO_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.k = k; p.v = v; p.g = g; p.S_loc = S_loc; p.G_tot = G_tot;
    BlockLayout w;
    if (!block_cut(w, d, ZECO_BLOCK_LOCAL_STATE, workspace, workspace_bytes)) return from_hip(launch_phase(p, d, 1, s));
    float *ws = static_cast<float *>(workspace);
    set_cut(p, cut_of(d->L, w.S));
    p.P = d->P * w.S;
    p.S_loc = ws; p.G_tot = ws + w.off_Gtot; p.pairs = 1;
    if (launch_phase(p, d, 1, s) != hipSuccess) return ZECO_ERR_HIP;
    zeco::ScanParams sp;
    fill_block_scan(sp, d, w.S);
    sp.S_loc = ws; sp.G_tot = ws + w.off_Gtot; sp.S_last = S_loc; sp.G_sum = G_tot; sp.pairs = 1;
    return from_hip(zeco::launch_scan(sp, s));
}

zeco_status zeco_gla_local_state(const zeco_gla_desc *d, const void *k, const void *v, const void *g,
                                 float *S_loc, float *G_tot, void *stream) {
    return zeco_gla_local_state_ws(d, k, v, g, S_loc, G_tot, nullptr, 0, stream);
}

zeco_status zeco_gla_fwd_from_state_ws(const zeco_gla_desc *d, const void *q, const void *k, const void *v,
                                       const void *g, const float *S_init, void *o, void *workspace,
                                       size_t workspace_bytes, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !S_init || !o) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(S_init) ||
        !aligned16(o))
        return ZECO_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    BlockLayout w;
    if (block_cut(w, d, ZECO_BLOCK_FWD_FROM_STATE, workspace, workspace_bytes)) {
        float *ws = static_cast<float *>(workspace);
        set_cut(p, cut_of(d->L, w.S));
        p.P = d->P * w.S;
        if (block_entering_states(p, w, ws, d, k, v, g, S_init, s) != hipSuccess) return ZECO_ERR_HIP;
        p.S_loc = nullptr; p.G_tot = nullptr;
        S_init = ws + w.off_Sinit;
    }
    p.q = q; p.k = k; p.v = v; p.g = g; p.o = o; p.S_init = S_init;
    return from_hip(launch_phase(p, d, 2, s));
}

zeco_status zeco_gla_fwd_from_state(const zeco_gla_desc *d, const void *q, const void *k, const void *v,
                                    const void *g, const float *S_init, void *o, void *stream) {
    return zeco_gla_fwd_from_state_ws(d, q, k, v, g, S_init, o, nullptr, 0, stream);
}

// The one-call forms treat the P segments as what they are together, one run of P * L tokens, and cut it into pieces
// of whole 64-token chunks as even as possible (Cut): where the pieces end is nobody's business but the library's,
// so neither the caller's segments nor a length without a small factor decide how many compute units work.  A piece
// is a workgroup's serial chain of chunks.  More pieces shorten the chain; each costs a prologue and its states
// (written by the first phase, scanned, read by the second), and a chunk takes the longer the more workgroups share
// the memory system.  The estimate, in microseconds, has two sets of constants, both fitted to sweeps of the piece count:
// for few (batch, head) pairs (d = 128, bf16, forward: 16 pairs x 16384 tokens, 8 / 16 / 32 pieces 152 / 138 / 152 us, 2048 tokens
// 42 (4) / 34 (8) / 36 (16) / 52 (32) us; training step over 131072 tokens, 12 / 16 / 32 pieces 3.34 / 3.04 / 3.15 ms), and for
// pairs that fill half of the compute units by themselves, where a piece's prologue and the last round of workgroups decide
// (256 pairs x 32768 tokens whole 2.34, in 2 3.70 ms; 640 x 16384 whole 3.15, in 2 4.64 ms; backward from saved states of 400 x
// 4096 in 1 / 3 / 4 / 16 pieces 1.93 / 1.89 / 1.98 / 2.30 ms).  The constants of the gradient passes (grad, bytesb) were fitted while dV was
// a pass of its own; the count picked takes 0.8 % (forward) and 1.0 % (training step) more than the best of up to 25 counts in the mean
// over 312 shapes of 1 .. 400 pairs, 11 and 17 % at worst, and 0.1 % of that is what a fit to the passes as they are would save.  A chain may
// be as long as it comes: 8 pairs x 2 M tokens in 32 / 256 pieces 7.12 / 7.30 ms forward (corrected: 4.85 / 5.65 ms), 16.6 / 16.5 ms backward.
struct PassCost {
    double chunk, bytes, hidden, start;   // a chunk's chain alone on the chip [us]; its traffic, divided by what of it is hidden; a piece's prologue and epilogue [us]
};
struct CostModel {
    PassCost one, two, grad;           // single pass, two phases, gradient passes
    double fixed1, fixed2, fixedb;
    double state;                      // bytes of a state
    double states2, statesb;           // states moved per piece
    double step2, stepb;               // of the scans, per piece
    double even, one_piece;            // factors in favour of equal pieces, and a margin for a single one
    double slots = kComputeUnits;      // workgroups in flight
    bool partial;                      // price a last round of fewer workgroups as such
    double second = 1.;                // a chunk's chain beside a second workgroup of the same compute unit
    bool bound = false;                // no chunk faster than its traffic at `rate`
    double rate = 5.9e6;               // bytes per microsecond of the chip
};
// `local`: for the passes of a cut local pass.
static CostModel cost_model(const zeco_gla_desc *d, long long pairs, bool local = false) {
    const bool f32 = d->io_dtype == ZECO_F32, wide = d->d_k == 128, many = pairs >= kComputeUnits / 2;
    const double io = f32 ? 4. : 2., k = io * d->d_k, v = io * d->d_v;
    const double g = d->g_per_head ? 4. : (d->g_dtype == ZECO_BF16 ? 2. : 4.) * d->d_k, f = (d->d_k * d->d_v) / 16384.;
    const double bytes1 = 64. * (2. * k + 2. * v + g), bytes2 = bytes1 + 64. * (k + v + g);
    const double bytesb = 64. * (9. * k + 8. * v + 3. * g + (d->g_per_head ? 12. : 12. * d->d_k));
    CostModel m;
    m.state = 4. * d->d_k * d->d_v;
    m.partial = many;
    if (many) {
        m.fixed1 = 5.; m.fixed2 = 9.5; m.fixedb = 7.2;
        m.states2 = 3.8; m.statesb = 4.5; m.step2 = m.stepb = 0.04;
        m.even = 0.97; m.one_piece = 1.;
    } else {
        m.fixed1 = 8.; m.fixed2 = 13.; m.fixedb = 30.;
        m.states2 = 6.; m.statesb = 7.; m.step2 = 0.07; m.stepb = 0.14;
        m.even = 0.92; m.one_piece = 0.93;
    }
    if (f32 && d->C != 16 && !local) {
        // 63 shapes of 1 .. 320 pairs, d = 64 and 128: the count picked takes 0.5 % more than the best of up to 17 in the mean, 8 % at worst
        m.fixed1 = 3.5; m.fixed2 = 11.; m.fixedb = 17.;
        m.states2 = 3.5; m.statesb = 8.; m.step2 = 0.045; m.stepb = 0.09;
        m.even = 0.97; m.one_piece = 1.;
        m.one = {3.3 + 8.1 * f, bytes1, 5.3, 0.};
        m.two = {5.3 + 11.1 * f, bytes2, 5.3, 0.};
        m.grad = {15.8 + 34. * f, bytesb, 4., f == 1. ? 15. : 0.};
        m.slots = 2. * kComputeUnits;
        m.second = 1.4;
        m.partial = true;
    } else if (f32 && many) {
        // (one workgroup on a compute unit: a second one takes as long again)
        m.one = {4.4 + 11. * f, bytes1, 5., 3.};
        m.two = {1.45 * (4. + 16. * f), bytes2, 5., 4. * f};
        m.grad = {1.45 * (12. + 41. * f), bytesb, 7., 25. * f};
    } else if (f32) {
        m.one = {4. + 13. * f, bytes1, 2.6, 0.};
        m.two = {6. + 20. * f, bytes2, 2.6, 0.};
        m.grad = {15. + 55. * f, bytesb, 2.6, 0.};
        m.slots = kComputeUnits * (d->C == 64 ? 1. : 2.);
    } else if (many) {
        m.one = {wide ? 1.9 : 1.15, bytes1, 1.75, 3.7 + 1.7 * f};
        m.two = {wide ? 2.6 : 1.65, bytes2, 1.83, 2. + 3.35 * f};
        m.grad = {wide ? 10.6 : 6.7, bytesb, 2.7, wide ? 14. : 2.5};
    } else {
        m.one = {wide ? 2.0 : 1.3, bytes1, 2.6, 0.};
        m.two = {wide ? 3.5 : 2.2, bytes2, 2.6, 0.};
        m.grad = {wide ? 13.5 : 9., bytesb, 2.6, 0.};
    }
    return m;
}
static double cost_chain(const CostModel &m, const PassCost &c, double wgs, double longest) {
    auto round = [&](double share) {
        const double traffic = share * c.bytes / m.rate;
        const double alone = c.chunk * (share > kComputeUnits ? m.second : 1.) + traffic / c.hidden;
        return c.start + longest * (m.bound && traffic > alone ? traffic : alone);
    };
    const double full = (double)(long long)(wgs / m.slots), rest = wgs - full * m.slots;
    if (rest <= 0.) return full * round(m.slots);
    return full * round(m.slots) + round(m.partial || full == 0. ? rest : m.slots);
}
static double cost_forward(const CostModel &m, double BH, double n, double longest, bool correct) {
    if (n == 1.) return m.fixed1 + cost_chain(m, m.one, BH, longest);
    // Pieces the AUTO schedule corrects instead of reading k, v, g twice: their first 35 chunks or so, what the decays of
    // a trained layer leave of a state, are then worked on again.
    const double part = correct ? (m.partial ? 0.55 + 12. / longest : 0.55 + 0.5 * 35. / longest) : 1.;
    return m.fixed2 + part * cost_chain(m, m.two, n * BH, longest) + m.states2 * n * BH * m.state / m.rate + m.step2 * n;
}
static double cost_backward(const CostModel &m, double BH, double n, double longest) {
    return m.fixedb + cost_chain(m, m.grad, n * BH, longest) + m.statesb * n * BH * m.state / m.rate + m.stepb * n;
}

// Does ZECO_SCHEDULE_AUTO take the correction?  It rounds o twice and its time depends on the decays (with decays near 1
// it is 15 - 20 % slower than two phases), so the cut must not bring calls to it: the caller's segments, halved while they
// halve evenly, stay within a round of workgroups and keep 256 tokens, have to be of 4096 tokens or more, and more than
// one (8 heads, 64 segments x 2048 tokens with decays near 1: two phases 0.47 ms, corrected in 32 pieces 0.51 ms) ..
static bool may_correct(const zeco_gla_desc *d) {
    if (d->io_dtype != ZECO_BF16) return false;
    const long long streams = (long long)d->B * d->P * d->H;
    int S = 1;
    auto halves_evenly = [&](int n) { return d->L % 64 == 0 ? d->L % (2 * n * 64) == 0 : d->L % (2 * n) == 0; };
    while (streams * S * 2 <= kComputeUnits && halves_evenly(S) && d->L / (2 * S) >= 256) S *= 2;
    return (long long)d->P * S > 1 && d->L / S >= 4096;
}
// .. and so the pieces of the cut (this many whole chunks).
static bool corrects(bool may, long long chunks) { return may && chunks >= 64; }

// Pieces per (batch, head).  Forward and backward share them, because the states the forward saves for the backward
// are the ones entering the pieces; the estimate weighs a backward a tenth (not every forward has one).  One
// piece, where the forward alone favours it: a single launch that reads everything once, and leaves the states of the
// pieces the backward then cuts for itself as it passes them.
static long long pieces_for(const zeco_gla_desc *d, long long T, bool backward, bool may_be_one = true) {
    const long long BH = (long long)d->B * d->H, chunks = T / 64;
    if (BH == 0) return 1;
    const CostModel m = cost_model(d, BH);
    const bool may = may_be_one && may_correct(d);   // (the calls over a table, which take two pieces at least, do not correct)
    const long long least = (chunks >> 22) + 1;      // (a piece's length is an int)
    long long best = 0, seen = 0;
    double cost = 0., cost_f = 0., cost_b = 0.;
    auto consider = [&](long long n) {
        if (n > chunks) n = chunks;
        if (n < 2 || n < least || n == seen || n == best || n * BH > (1ll << 24)) return;   // (the descriptor's limit on workgroups)
        seen = n;
        // (fp32 backward, C = 64: a second workgroup on a compute unit only for pieces of 512 tokens or more.  Over 72 shapes of 2 .. 64
        // heads the counts without this line take 0.91 of its time on geometric mean - 16 heads x 8192 tokens in 16 / 32 pieces, d = 64,
        // 247 / 205 us, d = 128, 522 / 483 - but up to 1.07: 24 x 8192, 128 x 64, 550 / 588, 4 x 8192, d = 128, 171 / 179)
        if (backward && m.second > 1. && d->C == 64 && n * BH > kComputeUnits && chunks / n < 8) return;
        const bool even = T % (64 * n) == 0;
        const double longest = (double)(chunks / n + (even ? 0 : 1));
        const double f = cost_forward(m, (double)BH, (double)n, longest, corrects(may, chunks / n)), b = cost_backward(m, (double)BH, (double)n, longest);
        // (equal pieces stay in step: 15 heads, 32768 tokens, 16 / 17 pieces 153 / 161 us)
        const double c = (backward ? b : f + 0.1 * b) * (even ? m.even : 1.);
        if (best == 0 || c < cost) { cost = c; cost_f = f; cost_b = b; best = n; }
    };
    // a quarter of the slots filled, .., four times over; the segments as they are, halved, ..; two to four chunks each, where
    // there are compute units for them, or eight and more
    for (int k : {1, 2, 3, 4, 6, 8, 12, 16}) consider(k * (long long)m.slots / (4 * BH));
    for (long long n = d->P; n <= chunks && n * BH <= 4 * (long long)m.slots; n *= 2) consider(n);
    if (BH < kComputeUnits) for (int k = 2; k <= 4; ++k) consider((chunks + k - 1) / k);
    if (m.partial) for (long long n = 2; n <= chunks / 8; n *= 2) consider(n);
    if (may) consider(chunks / 64);   // just enough for the correction
    if (least == 1 && may_be_one) {
        const double whole = m.second > 1. ? (double)T / 64. : (double)chunks;
        const double one = backward ? cost_backward(m, (double)BH, 1., whole) : cost_forward(m, (double)BH, 1., whole, false);
        if (best == 0 || one <= m.one_piece * (backward ? cost_b : cost_f)) best = 1;
    }
    return best ? best : least;
}

// Number of sub-segments each segment is cut into inside zeco_gla_local_fwd (1 = none).  A stream is
// a serial chain over chunks, so with few (batch, segment, head) streams most compute units would
// idle; the local pass then applies the method to itself: sub-segment states from the zero state, a scan
// of them inside each segment, and the output pass of every sub-segment from its scanned state.  Sub-segments of at
// least 256 tokens, in one round of workgroups; how many, by the estimate of the one-call forms (the cut need not
// come out even: 5 x 2 streams of 7133 tokens took one workgroup pair each before).
static int subsegments(const zeco_gla_desc *d) {
    const long long streams = (long long)d->B * d->P * d->H, chunks = d->L / 64;
    if (streams > 64 || streams == 0) return 1;
    CostModel m = cost_model(d, streams, true);
    m.two.bytes += 64. * (d->g_per_head ? 4. : 4. * d->d_k);   // G_cum
    m.bound = true;   // (three calls, 6 heads, 2 x 32768 tokens, 16 / 21 sub-segments: 285 / 302 us)
    long long best = 1;
    double cost = 0.;
    auto consider = [&](long long S) {
        if (S * 4 > chunks) S = chunks / 4;
        if (S < 2 || S * streams > kComputeUnits) return;
        const bool even = d->L % (64 * S) == 0;
        const double c = cost_forward(m, (double)streams, (double)S, (double)(d->L / 64 / S + (even ? 0 : 1)), false) * (even ? 0.92 : 1.);
        if (best == 1 || c < cost) { cost = c; best = S; }
    };
    for (int k = 2; k <= 4; ++k) consider(64 * k / streams);
    for (long long S = 2; S * streams <= kComputeUnits; S *= 2) consider(S);
    return (int)best;
}

// Pieces per segment of a building block (1: the segments are run whole), by an estimate in microseconds like the one above.
// A whole segment costs whole + n chunks of (whole_chunk + what of the pass's traffic is not hidden), S pieces of it cut + the
// same per chunk of the longest piece (the pass that makes the states included) + the scan.  Beyond 128 workgroups (256 for the
// fp32 kernels at C = 32 and 64, two of which share a compute unit) a chunk's chain counts `alone` times: the bf16 passes stop splitting
// a stream over siblings there.  The constants are a fit and stand together - of the kernels without siblings some have `alone` below
// one, which takes back what `chunk` and the traffic term overstate - to 360 measurements of each call (2 .. 128 streams of 512 .. 8192
// tokens, 1 .. 128 pieces; 3 - 8 % off in the mean); the count picked takes 0.7 % more than the best one on average, 19 % at worst.
// More than 128 streams were not measured and are not cut.  64 streams x 8192 tokens, d = 128, whole -> in 4: states 171 -> 92, output pass 322 -> 226, state gradients 177 ->
// 96, gradients 1193 -> 635 us; 16 x 2048 in 8: 38 -> 15, 73 -> 33, 38 -> 14, 255 -> 76; 128 x 8192 in 2: 194 -> 169, 371 whole, 197 -> 178,
// 1342 -> 1231.
struct BlockCost { double whole, cut, whole_chunk, chunk, hidden, step, states, alone; };
static int block_pieces(const zeco_gla_desc *d, int call) {
    static const BlockCost cost[4][5] = {   // by call; d = 128, smaller heads, one decay per head, fp32 at C = 16, fp32
        {{3.5, 7.7, 1.02, 0.95, 2.96, 0.083, 1.8, 1.62}, {3.2, 7.5, 1.11, 1.01, 6.0, 0.08, 2.5, 1.08},
         {4.7, 7.8, 0.72, 0.70, 2.4, 0.074, 2.2, 1.5}, {4.8, 5.9, 5.2, 5.6, 1.41, 0.03, 2.6, 0.76},
         {3.8, 6.9, 5.8, 5.85, 3.6, 0.064, 2., 1.27}},
        {{4.7, 12.5, 2.12, 3.05, 4.0, 0.08, 3.4, 1.48}, {3.9, 9.9, 1.43, 2.55, 4.8, 0.11, 5.4, 1.06},
         {5.6, 13.2, 1.72, 2.5, 4.7, 0.085, 3.2, 1.5}, {2.9, 2.5, 13., 19.1, 1.21, 0., 7.8, 0.73},
         {1.9, 8.6, 11.6, 17.6, 6., 0.053, 5.2, 1.36}},
        {{2.9, 7.7, 1.05, 0.98, 3.0, 0.04, 1.5, 1.68}, {2.7, 7.1, 1.17, 1.1, 6.1, 0.034, 2.5, 1.05},
         {4.7, 7.8, 0.72, 0.70, 2.2, 0.026, 1.85, 1.46}, {4.1, 5.2, 5.35, 5.6, 1.38, 0., 2.7, 0.72},
         {3.1, 6.1, 6.1, 6.1, 5., 0.023, 2.2, 1.32}},
        {{6., 26.1, 7.7, 8.4, 3.3, 0.17, 6.7, 1.35}, {7.3, 20., 5.2, 6.5, 3.5, 0.21, 12., 0.91},
         {13., 29.8, 7.7, 9.0, 5.05, 0.18, 5.6, 1.08}, {18.5, 16., 38.5, 51.2, 1.05, 0.04, 12., 0.78},
         {1.6, 18.7, 40.2, 52., 3.4, 0.094, 12., 1.34}}};
    const long long streams = (long long)d->B * d->P * d->H, chunks = d->L / 64;
    if (streams > kComputeUnits / 2 || streams == 0 || chunks < 8) return 1;
    const bool f32 = d->io_dtype == ZECO_F32, x3 = f32 && d->C != 16;   // (two workgroups a compute unit, no siblings)
    const BlockCost &m = cost[call][x3 ? 4 : f32 ? 3 : d->g_per_head ? 2 : d->d_k == 128 && d->d_v == 128 ? 0 : 1];
    const double io = f32 ? 4. : 2., k = io * d->d_k, v = io * d->d_v, rate = 5.9e6;
    const double g = d->g_per_head ? 4. : (d->g_dtype == ZECO_BF16 ? 2. : 4.) * d->d_k, dg = d->g_per_head ? 4. : 4. * d->d_k;
    const double states = 64. * (k + v + g);
    const double pass = call == ZECO_BLOCK_FWD_FROM_STATE ? 64. * (2. * k + 2. * v + g)
                        : call == ZECO_BLOCK_BWD_FROM_STATE ? 64. * (7. * k + 5. * v + 3. * g + 3. * dg) : states;
    const double both = pass == states ? states : states + pass;
    const double slots = (double)kComputeUnits * (f32 ? 2. : 1.), size = x3 ? 0.3 + 0.7 * d->d_k * d->d_v / 16384. : 1.;
    auto per_chunk = [&](double chunk, double wgs, double bytes) {
        return size * chunk * (wgs > kComputeUnits / (x3 ? 1 : 2) ? m.alone : 1.) + wgs * bytes / (rate * m.hidden);
    };
    long long best = 1;
    double least = 0.95 * (m.whole + (double)((d->L + 63) / 64) * per_chunk(m.whole_chunk, (double)streams, pass));
    auto consider = [&](long long S) {
        if (S > chunks) S = chunks;
        const double wgs = (double)S * streams;
        if (S < 2 || wgs > slots) return;
        const bool even = d->L % (64 * S) == 0;
        const double t = (m.cut + m.step * S + m.states * wgs * 4. * d->d_k * d->d_v / rate +
                          (double)(chunks / S + (even ? 0 : 1)) * per_chunk(m.chunk, wgs, both)) * (even ? 0.97 : 1.);
        if (t < least) { least = t; best = S; }
    };
    for (int j = 1; j <= 4; ++j) consider((long long)slots * j / (4 * streams));
    for (long long S = 2; S * streams <= slots; S *= 2) consider(S);
    for (int j = 1; j <= 3; ++j) consider((chunks + j - 1) / j);
    return (int)best;
}

// The cut itself, and what the launches need to know of it.
static zeco::Cut cut_of(long long tokens, long long n) {
    zeco::Cut c;
    c.n = (int)n; c.base = (int)(tokens / 64 / n); c.rem = (int)(tokens / 64 % n); c.len = tokens;
    return c;
}
static int longest_chunks(const zeco::Cut &c) {
    const int tail = (c.len & 63) ? 1 : 0;
    return c.base + (c.rem == 0 ? tail : 1);   // (rem < n: the first piece, which has the tail, is one of base chunks)
}
static int longest_tokens(const zeco::Cut &c) {   // upper bound of the pieces' lengths
    return c.rem ? 64 * (c.base + 1) : 64 * c.base + (int)(c.len & 63);
}
// Equal pieces of whole chunks are segments like any others, and the launches take them as such: working a piece out cost
// 0.2 - 0.4 us a launch (16 heads x 16384 tokens, three launches: 130.9 -> 130.2 us; per-head training step, 16 heads x
// 8 x 4096 tokens, six: 694 -> 691 us).
static bool equal_pieces(const zeco::Cut &c) { return c.rem == 0 && (c.len & 63) == 0; }
static void set_cut(zeco::ChunkParams &p, const zeco::Cut &c) {
    p.P = c.n;
    if (equal_pieces(c)) { set_length(p, longest_tokens(c)); return; }
    p.cut = c; p.n_chunks = longest_chunks(c); p.pad = 0;
}

// Workspace of zeco_gla_fused_fwd, in floats: piece states S_loc [n], S_init [n], their G_tot [n], the
// cumulative decay of the CORRECT schedule (per chunk and channel, or per token with per-head gates), and
// the scratch of the piece scan where it runs as a tree.
struct FwdLayout {
    size_t n, states, off_Sinit, off_Gtot, off_decay, off_tree, total;
};
static FwdLayout fwd_layout(const zeco_gla_desc *d, const zeco::Cut &cut) {
    FwdLayout w;
    const size_t gd = d->g_per_head ? 1 : d->d_k;
    w.n = (size_t)cut.n * d->B * d->H;
    w.states = w.n * d->d_k * d->d_v;
    w.off_Sinit = w.states;
    w.off_Gtot = 2 * w.states;
    w.off_decay = w.off_Gtot + ((w.n * gd + 3) & ~(size_t)3);
    const size_t decay = d->g_per_head ? (size_t)d->B * d->P * d->L * d->H
                                       : (size_t)d->B * cut.n * longest_chunks(cut) * d->H * d->d_k;
    w.off_tree = w.off_decay + ((decay + 3) & ~(size_t)3);
    w.total = w.off_tree + chain_scratch_floats(cut.n, d->B * d->H, d->d_k, d->d_v, d->g_per_head);
    return w;
}
static zeco::Cut fwd_cut(const zeco_gla_desc *d) { const long long T = (long long)d->P * d->L; return cut_of(T, pieces_for(d, T, false)); }
static zeco::Cut bwd_cut(const zeco_gla_desc *d) {
    const zeco::Cut c = fwd_cut(d);
    const bool own = d->io_dtype == ZECO_F32 && d->C != 16;   // (an fp32 forward saves no states: each direction takes its own count)
    return c.n > 1 && !own ? c : cut_of(c.len, pieces_for(d, c.len, true));
}

size_t zeco_gla_fused_fwd_workspace(const zeco_gla_desc *desc) {
    if (check_desc(desc, true) != ZECO_OK) return 0;
    return fwd_layout(desc, fwd_cut(desc)).total * sizeof(float);
}

zeco_status zeco_gla_fused_fwd(const zeco_gla_desc *d, const void *q, const void *k, const void *v,
                               const void *g, const float *S0, void *o, float *S_last, float *S_save,
                               int32_t schedule, void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !o || !workspace) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(o) ||
        !aligned16(S0) || !aligned16(S_last) || !aligned16(S_save) || !aligned16(workspace))
        return ZECO_ERR_INVALID_ARG;
    if (schedule != ZECO_SCHEDULE_AUTO && schedule != ZECO_SCHEDULE_TWO_PHASE && schedule != ZECO_SCHEDULE_CORRECT)
        return ZECO_ERR_INVALID_ARG;
    // fp32: the two phases of Alg. 1 only (no chunk-decay correction, no states saved for a backward)
    if (d->io_dtype != ZECO_BF16 && S_save) return ZECO_ERR_UNSUPPORTED;
    const bool can_correct = d->io_dtype == ZECO_BF16;
    if (schedule == ZECO_SCHEDULE_CORRECT && !can_correct) return ZECO_ERR_UNSUPPORTED;
    const zeco::Cut cut = fwd_cut(d);
    const FwdLayout w = fwd_layout(d, cut);
    if (workspace_bytes < w.total * sizeof(float)) return ZECO_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    float *Sloc = static_cast<float *>(workspace), *Sinit = Sloc + w.off_Sinit, *Gtot = Sloc + w.off_Gtot;
    float *Gchunk = Sloc + w.off_decay, *tree = Sloc + w.off_tree;
    // With S_save the scan writes the states entering the pieces, and the end state after them, straight into
    // it: the backward works on the same pieces and reads them there (S_save [n pieces + 1 slot per (b, h)]).
    if (S_save) Sinit = S_save;
    float *save_last = S_save ? S_save + w.states : nullptr;

    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    set_cut(p, cut);
    hipError_t e;
    if (cut.n == 1) {
        // one piece per (batch, head): the state entering it is S0, so the output pass alone does it all and leaves the
        // end state, and the states entering the backward's pieces, on its way (the first phase, its scan and a second
        // read of k, v, g would be for nothing)
        p.q = q; p.k = k; p.v = v; p.g = g; p.o = o;
        p.S_init = S0; p.S_loc = S_last;
        if (S_save) {
            p.emit = bwd_cut(d);
            p.S_emit = S_save; p.S_loc2 = S_save + (size_t)p.emit.n * d->B * d->H * d->d_k * d->d_v;
        }
        return from_hip(launch_phase(p, d, d->io_dtype == ZECO_F32 ? 2 : 7, s));
    }
    const bool correct = schedule == ZECO_SCHEDULE_CORRECT || (schedule == ZECO_SCHEDULE_AUTO && corrects(may_correct(d), cut.base));

    // first pass: the pieces from the zero state - with their local outputs and the cumulative decay per chunk
    // (per token with per-head gates, whose G_cum is 4 bytes per token and head), or their end states only
    p.k = k; p.v = v; p.g = g; p.S_loc = Sloc; p.G_tot = Gtot;
    if (correct) {
        p.q = q; p.o = o;
        if (d->g_per_head) p.G_cum = Gchunk; else p.G_chunk = Gchunk;
        e = zeco::launch_chunk_bf16(p, d->d_k, d->d_v, chunk_gate(d), d->g_per_head ? 0 : 6, s);
    } else {
        e = launch_phase(p, d, 1, s);
    }
    if (e != hipSuccess) return ZECO_ERR_HIP;

    zeco::ScanParams sp;
    sp.S_loc = Sloc; sp.G_tot = Gtot; sp.S0 = S0; sp.S_init = Sinit; sp.S_last = S_save ? save_last : S_last;
    sp.S_last2 = S_save ? S_last : nullptr;   // (by the scan, not a copy of its own: 16 heads, d = 128, 2.4 us and a launch)
    sp.P = p.P; sp.groups = 1; sp.BH = d->B * d->H; sp.d_k = d->d_k; sp.d_v = d->d_v;
    sp.rows_per_block = d->d_k / 16; sp.gate_per_head = d->g_per_head;
    if ((e = launch_scan_chain(sp, tree, s)) != hipSuccess) return ZECO_ERR_HIP;

    if (correct) {   // correction of the pieces' heads
        zeco::ApplyParams ap;
        fill_apply_params(ap, d, p.P, longest_tokens(cut));
        if (!equal_pieces(cut)) {
            ap.cut = cut; ap.n_chunks = longest_chunks(cut); ap.pad = 0;
            set_apply_share(ap, longest_tokens(cut), 1024, false);
        }
        ap.q = q; ap.S_init = Sinit; ap.o = o;
        ap.p0 = S0 ? 0 : 1;
        if (d->g_per_head) {
            ap.G_cum = Gchunk;
            return from_hip(zeco::launch_apply_bf16(ap, d->d_k, d->d_v, s));
        }
        ap.g = g; ap.g_bf16 = d->g_dtype == ZECO_BF16; ap.G_chunk = Gchunk;
        return from_hip(zeco::launch_apply_cd_bf16(ap, d->d_k, d->d_v, s));
    }
    p.q = q; p.o = o; p.S_init = Sinit; p.S_loc = nullptr; p.G_tot = nullptr;   // output pass from the scanned states
    return from_hip(launch_phase(p, d, 2, s));
}

// ---- backward (App. A.4) ------------------------------------------------------------------------------
// The gradient passes over `P` pieces of `L` tokens.  dQ from the forward states; with `dS_loc` it also
// emits every piece's state gradient from dS = 0 (and with `G_tot_out` its total log decay), which is
// what the reverse scan chains into dS_in.
// `cut` null: the segments as they are; otherwise P counts its pieces and L bounds their lengths.
static void fill_bwd_params(zeco::BwdQKParams &b, const zeco_gla_desc *d, int P, int L, const void *g,
                            float *dg, const float *S_init, const float *S_last, const zeco::Cut *cut) {
    if (cut && !equal_pieces(*cut)) b.cut = *cut;
    b.T = (long long)d->P * d->L;
    b.g = g; b.B = d->B; b.P = P; b.H = d->H; b.L = L; b.n_chunks = chunks_of(L); b.pad = 64 * b.n_chunks - L;
    b.sb = d->stride_b; b.st = d->stride_t; b.sh = d->stride_h;
    b.vb = d->vstride_b; b.vt = d->vstride_t; b.vh = d->vstride_h;
    b.dg = dg; b.S_init = S_init; b.S_last = S_last;
}

// Checkpoints of the forward state per (batch, segment, head) that re-anchor dG: one at every 8th chunk
// boundary inside a segment of (at most) L tokens.
static int bwd_checkpoints(int L) { return (chunks_of(L) - 1) / 8; }
static size_t bwd_checkpoint_floats(const zeco_gla_desc *d, int P, int L) {
    return (size_t)d->B * P * d->H * bwd_checkpoints(L) * d->d_k * d->d_v;
}

static zeco_status bwd_dq_pass(const zeco_gla_desc *d, int P, int L, const void *q, const void *k,
                               const void *v, const void *g, const void *dO, const float *S_init,
                               const float *S_last, void *dq, float *dg, float *dS_loc, float *G_tot_out,
                               float *S_ck, hipStream_t s, const int64_t *seg_start = nullptr, int64_t T = 0,
                               const zeco::Cut *cut = nullptr, int plan = 0) {
    zeco::BwdQKParams b;
    fill_bwd_params(b, d, P, L, g, dg, S_init, S_last, cut);
    if (S_ck && bwd_checkpoints(L) > 0) { b.S_ck = S_ck; b.n_ck = bwd_checkpoints(L); b.short_last = 1; }
    if (seg_start) { b.seg_start = reinterpret_cast<const long long *>(seg_start); b.T = T; b.plan = plan; }
    b.x = dO; b.y = v; b.z = k; b.z2 = q; b.out = dq; b.W_init = S_init; b.zscale = 1.f; b.oscale = d->scale;
    if (d->io_dtype == ZECO_F32) {
        // the fp32 kernels: dQ, and the segments' state gradients from dS = 0 as a pass of their own
        if (zeco::launch_bwd_qk_f32(b, d->d_k, d->d_v, d->C, false, s) != hipSuccess) return ZECO_ERR_HIP;
        if (!dS_loc) return ZECO_OK;
        zeco::ChunkParams c;
        fill_chunk_params(c, d);
        set_length(c, L);
        if (cut) set_cut(c, *cut);
        c.P = P;   // (pieces of all runs)
        if (seg_start) { c.seg_start = reinterpret_cast<const long long *>(seg_start); c.T = T; c.plan = plan; }
        c.k = q; c.v = dO; c.g = g; c.S_loc = dS_loc; c.G_tot = G_tot_out; c.scale = 1.f; c.kscale = d->scale;
        return from_hip(launch_phase(c, d, 3, s));
    }
    b.dS_loc = dS_loc; b.G_tot_out = G_tot_out; b.qscale = d->scale;
    return from_hip(zeco::launch_bwd_qk(b, d->d_k, d->d_v, gate_mode(d), false, s));
}

// dV and dK from the state gradients entering the pieces, dG from all of them (after the dQ pass, whose
// q .* dq left in dg the dK pass consumes).
static zeco_status bwd_dv_dk_passes(const zeco_gla_desc *d, int P, int L, const void *q, const void *k,
                                    const void *v, const void *g, const void *dO, const float *S_init,
                                    const float *S_last, const float *dS_in, void *dk, void *dv,
                                    float *dg, float *S_ck, hipStream_t s, const int64_t *seg_start = nullptr,
                                    int64_t T = 0, const zeco::Cut *cut = nullptr, int plan = 0) {
    if (d->io_dtype == ZECO_F32) {
        zeco::ChunkParams c;
        fill_chunk_params(c, d);
        set_length(c, L);
        if (cut) set_cut(c, *cut);
        c.P = P;   // (pieces of all runs)
        if (seg_start) { c.seg_start = reinterpret_cast<const long long *>(seg_start); c.T = T; c.plan = plan; }
        c.q = k; c.k = q; c.v = dO; c.g = g; c.o = dv; c.S_init = dS_in; c.scale = 1.f; c.kscale = d->scale;
        if (launch_phase(c, d, 4, s) != hipSuccess) return ZECO_ERR_HIP;
    }
    zeco::BwdQKParams b;
    fill_bwd_params(b, d, P, L, g, dg, S_init, S_last, cut);
    if (seg_start) { b.seg_start = reinterpret_cast<const long long *>(seg_start); b.T = T; b.plan = plan; }
    b.x = v; b.y = dO; b.z = q; b.z2 = k; b.out = dk; b.out2 = dv; b.W_init = dS_in; b.zscale = d->scale; b.oscale = 1.f;
    if (S_ck && bwd_checkpoints(L) > 0) { b.S_ck = S_ck; b.n_ck = bwd_checkpoints(L); }
    if (d->io_dtype == ZECO_F32) return from_hip(zeco::launch_bwd_qk_f32(b, d->d_k, d->d_v, d->C, true, s));
    return from_hip(zeco::launch_bwd_qk(b, d->d_k, d->d_v, gate_mode(d), true, s));   // (dV in the same pass)
}

zeco_status zeco_gla_bwd_dstate_ws(const zeco_gla_desc *d, const void *q, const void *g, const void *dO, float *dS_loc,
                                   void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !g || !dO || !dS_loc) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(g) || !aligned16(dO) || !aligned16(dS_loc)) return ZECO_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.k = q; p.v = dO; p.g = g; p.S_loc = dS_loc; p.kscale = d->scale;
    BlockLayout w;
    if (!block_cut(w, d, ZECO_BLOCK_BWD_DSTATE, workspace, workspace_bytes)) return from_hip(launch_phase(p, d, 3, s));
    float *ws = static_cast<float *>(workspace);
    set_cut(p, cut_of(d->L, w.S));
    p.P = d->P * w.S;
    p.S_loc = ws; p.G_tot = ws + w.off_Gtot;
    if (launch_phase(p, d, 3, s) != hipSuccess) return ZECO_ERR_HIP;
    zeco::ScanParams sp;
    fill_block_scan(sp, d, w.S);
    sp.S_loc = ws; sp.G_tot = ws + w.off_Gtot; sp.S_last = dS_loc; sp.reverse = 1;
    return from_hip(zeco::launch_scan(sp, s));
}

zeco_status zeco_gla_bwd_dstate(const zeco_gla_desc *d, const void *q, const void *g, const void *dO,
                                float *dS_loc, void *stream) {
    return zeco_gla_bwd_dstate_ws(d, q, g, dO, dS_loc, nullptr, 0, stream);
}

size_t zeco_gla_bwd_from_state_workspace(const zeco_gla_desc *desc) {
    if (check_desc(desc, true) != ZECO_OK) return 0;
    return bwd_checkpoint_floats(desc, desc->P, desc->L) * sizeof(float);
}

// `may_cut`: the _ws form, which takes more than its checkpoints' workspace for leave to cut the segments (the other one never
// writes past its own size, however much it is given).
static zeco_status bwd_from_state(const zeco_gla_desc *d, const void *q, const void *k, const void *v, const void *g, const void *dO,
                                  const float *S_init, const float *S_last, const float *dS_in, void *dq, void *dk, void *dv,
                                  float *dg, void *workspace, size_t workspace_bytes, void *stream, bool may_cut) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    const size_t need = zeco_gla_bwd_from_state_workspace(d);
    if (workspace_bytes < need) return ZECO_ERR_WORKSPACE;
    if (need && (!workspace || !aligned16(workspace))) return ZECO_ERR_INVALID_ARG;
    if (!q || !k || !v || !g || !dO || !S_init || !S_last || !dS_in || !dq || !dk || !dv || !dg)
        return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(dO) ||
        !aligned16(S_init) || !aligned16(S_last) || !aligned16(dS_in) || !aligned16(dq) || !aligned16(dk) ||
        !aligned16(dv) || !aligned16(dg))
        return ZECO_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    BlockLayout w;
    if (may_cut && block_cut(w, d, ZECO_BLOCK_BWD_FROM_STATE, workspace, workspace_bytes)) {
        // as in zeco_gla_fused_bwd, with the states and gradients entering the segments given: forward states of the
        // pieces, dQ with the pieces' state gradients, their scan inside the segments, dK, dV and dG
        float *ws = static_cast<float *>(workspace), *Sin = ws + w.off_Sinit, *dSin = ws + w.off_dSin;
        const zeco::Cut cut = cut_of(d->L, w.S);
        const int P = d->P * w.S, L = longest_tokens(cut);
        zeco::ChunkParams p;
        fill_chunk_params(p, d);
        set_cut(p, cut);
        p.P = P;
        if (block_entering_states(p, w, ws, d, k, v, g, S_init, s) != hipSuccess) return ZECO_ERR_HIP;
        float *S_ck = bwd_checkpoints(L) > 0 ? ws + w.off_ck : nullptr;
        zeco_status zs = bwd_dq_pass(d, P, L, q, k, v, g, dO, Sin, S_last, dq, dg, ws, ws + w.off_Gtot, S_ck, s, nullptr, 0, &cut);
        if (zs != ZECO_OK) return zs;
        zeco::ScanParams sp;
        fill_block_scan(sp, d, w.S);
        sp.S_loc = ws; sp.G_tot = ws + w.off_Gtot; sp.S0 = dS_in; sp.S_init = dSin; sp.reverse = 1;
        if (zeco::launch_scan(sp, s) != hipSuccess) return ZECO_ERR_HIP;
        return bwd_dv_dk_passes(d, P, L, q, k, v, g, dO, Sin, S_last, dSin, dk, dv, dg, S_ck, s, nullptr, 0, &cut);
    }
    float *S_ck = need ? static_cast<float *>(workspace) : nullptr;
    const zeco_status sq = bwd_dq_pass(d, d->P, d->L, q, k, v, g, dO, S_init, S_last, dq, dg, nullptr, nullptr, S_ck, s);
    if (sq != ZECO_OK) return sq;
    return bwd_dv_dk_passes(d, d->P, d->L, q, k, v, g, dO, S_init, S_last, dS_in, dk, dv, dg, S_ck, s);
}

zeco_status zeco_gla_bwd_from_state(const zeco_gla_desc *d, const void *q, const void *k, const void *v,
                                    const void *g, const void *dO, const float *S_init, const float *S_last,
                                    const float *dS_in, void *dq, void *dk, void *dv, float *dg,
                                    void *workspace, size_t workspace_bytes, void *stream) {
    return bwd_from_state(d, q, k, v, g, dO, S_init, S_last, dS_in, dq, dk, dv, dg, workspace, workspace_bytes, stream, false);
}

zeco_status zeco_gla_bwd_from_state_ws(const zeco_gla_desc *d, const void *q, const void *k, const void *v,
                                       const void *g, const void *dO, const float *S_init, const float *S_last,
                                       const float *dS_in, void *dq, void *dk, void *dv, float *dg,
                                       void *workspace, size_t workspace_bytes, void *stream) {
    return bwd_from_state(d, q, k, v, g, dO, S_init, S_last, dS_in, dq, dk, dv, dg, workspace, workspace_bytes, stream, true);
}

// zeco_gla_fused_bwd works on the forward's pieces (bwd_cut), whose entering states the forward can save for it.  The
// gate gradient, a running sum of nearly cancelling terms whose bf16 rounding noise grows with the square root of
// the run length, is re-anchored every 512 tokens inside a piece from the forward-state checkpoints of the dQ pass, so
// the pieces need not be short for its sake: cut down to 512 tokens each the same passes spend 12-20 % more time on
// pipeline prologues, on the states of many more pieces and on scans over them.

// Workspace of zeco_gla_fused_bwd, in floats: forward piece states S_loc [n], S_init [n + one more
// slot per (b,h) for the final state], their G_tot [n]; state gradients dS_loc [n], dS_in [n].
struct BwdLayout {
    size_t n, state, off_Sloc, off_Sinit, off_Gtot, off_dSloc, off_dSin, off_tree, off_ck, total;
};
static BwdLayout bwd_layout(const zeco_gla_desc *d, const zeco::Cut &cut) {
    BwdLayout w;
    const size_t bh = (size_t)d->B * d->H;
    w.n = (size_t)cut.n * bh;
    w.state = (size_t)d->d_k * d->d_v;
    w.off_Sloc = 0;
    w.off_Sinit = w.off_Sloc + w.n * w.state;
    w.off_Gtot = w.off_Sinit + (w.n + bh) * w.state;
    w.off_dSloc = w.off_Gtot + w.n * d->d_k;
    w.off_dSin = w.off_dSloc + w.n * w.state;
    w.off_tree = w.off_dSin + w.n * w.state;   // scratch of the two piece scans where they run as trees
    w.off_ck = w.off_tree + chain_scratch_floats(cut.n, d->B * d->H, d->d_k, d->d_v, d->g_per_head);
    w.total = w.off_ck + bwd_checkpoint_floats(d, cut.n, longest_tokens(cut));   // checkpoints inside the pieces
    return w;
}

size_t zeco_gla_saved_states_bytes(const zeco_gla_desc *desc) {
    if (check_desc(desc, true) != ZECO_OK || desc->io_dtype != ZECO_BF16) return 0;
    return ((size_t)bwd_cut(desc).n + 1) * desc->B * desc->H * desc->d_k * desc->d_v * sizeof(float);
}

size_t zeco_gla_fused_bwd_workspace(const zeco_gla_desc *desc) {
    if (check_desc(desc, true) != ZECO_OK) return 0;
    return bwd_layout(desc, bwd_cut(desc)).total * sizeof(float);
}

zeco_status zeco_gla_fused_bwd(const zeco_gla_desc *d, const void *q, const void *k, const void *v,
                               const void *g, const void *dO, const float *S0, const float *dS_T,
                               const float *S_saved, void *dq, void *dk, void *dv, float *dg, float *dS0,
                               void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !dO || !dq || !dk || !dv || !dg || !workspace) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(dO) ||
        !aligned16(S0) || !aligned16(dS_T) || !aligned16(S_saved) || !aligned16(dq) || !aligned16(dk) || !aligned16(dv) ||
        !aligned16(dg) || !aligned16(dS0) || !aligned16(workspace))
        return ZECO_ERR_INVALID_ARG;
    if (d->io_dtype != ZECO_BF16 && S_saved) return ZECO_ERR_UNSUPPORTED;   // (the fp32 forward saves no states)
    const zeco::Cut cut = bwd_cut(d);
    const BwdLayout w = bwd_layout(d, cut);
    if (workspace_bytes < w.total * sizeof(float)) return ZECO_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    float *ws = static_cast<float *>(workspace);
    float *Sloc = ws + w.off_Sloc, *Sinit = ws + w.off_Sinit, *Gtot = ws + w.off_Gtot;
    float *dSloc = ws + w.off_dSloc, *dSin = ws + w.off_dSin;
    float *Slast = Sinit + w.n * w.state;
    const int P = cut.n, L = longest_tokens(cut);

    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    set_cut(p, cut);
    zeco::ScanParams sp;
    sp.P = P; sp.groups = 1; sp.BH = d->B * d->H; sp.d_k = d->d_k; sp.d_v = d->d_v;
    sp.rows_per_block = d->d_k / 16; sp.gate_per_head = d->g_per_head;
    hipError_t e;
    const float *Sin = Sinit, *Sl = Slast;
    if (S_saved) {
        // forward states at the piece boundaries as the forward left them
        Sin = S_saved; Sl = S_saved + w.n * w.state;
    } else {
        // recomputed: phase 1 of the forward and its scan
        p.k = k; p.v = v; p.g = g; p.S_loc = Sloc; p.G_tot = Gtot;
        if ((e = launch_phase(p, d, 1, s)) != hipSuccess) return ZECO_ERR_HIP;
        sp.S_loc = Sloc; sp.G_tot = Gtot; sp.S0 = S0; sp.S_init = Sinit; sp.S_last = Slast;
        if ((e = launch_scan_chain(sp, ws + w.off_tree, s)) != hipSuccess) return ZECO_ERR_HIP;
    }

    // dQ from the forward states; the same pass leaves every piece's state gradient from dS = 0 (and
    // the pieces' total decays when the forward state pass did not run), which the reverse scan chains
    // from the last piece to the first
    float *S_ck = bwd_checkpoints(L) > 0 ? ws + w.off_ck : nullptr;
    zeco_status zs = bwd_dq_pass(d, P, L, q, k, v, g, dO, Sin, Sl, dq, dg, dSloc, S_saved ? Gtot : nullptr, S_ck, s,
                                 nullptr, 0, &cut);
    if (zs != ZECO_OK) return zs;
    sp.S_loc = dSloc; sp.G_tot = Gtot; sp.S0 = dS_T; sp.S_init = dSin; sp.S_last = dS0; sp.reverse = 1;
    if ((e = launch_scan_chain(sp, ws + w.off_tree, s)) != hipSuccess) return ZECO_ERR_HIP;

    return bwd_dv_dk_passes(d, P, L, q, k, v, g, dO, Sin, Sl, dSin, dk, dv, dg, S_ck, s, nullptr, 0, &cut);
}

zeco_status zeco_state_scan(int32_t P, int32_t BH, int32_t d_k, int32_t d_v, int32_t K_blocks,
                            const float *S_loc, const float *G_tot, const float *S0, float *S_init,
                            float *S_last, int32_t direction, int32_t gate_per_head, void *stream) {
    if (P <= 0 || BH < 0 || d_k <= 0 || d_v <= 0 || K_blocks <= 0) return ZECO_ERR_INVALID_ARG;
    if (d_k % K_blocks != 0) return ZECO_ERR_INVALID_ARG;
    if (direction != 0 && direction != 1) return ZECO_ERR_INVALID_ARG;
    if (gate_per_head != 0 && gate_per_head != 1) return ZECO_ERR_INVALID_ARG;
    if (BH == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!S_loc || !G_tot || !S_init) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(S_loc) || !aligned16(S_init) || !aligned16(S0) || !aligned16(S_last) ||
        (reinterpret_cast<uintptr_t>(G_tot) & 3u))
        return ZECO_ERR_INVALID_ARG;
    if ((int64_t)BH * K_blocks > (int64_t)1 << 30) return ZECO_ERR_INVALID_ARG;
    if (d_v % 4 != 0) return ZECO_ERR_UNSUPPORTED;

    zeco::ScanParams p;
    p.reverse = direction; p.gate_per_head = gate_per_head;
    p.S_loc = S_loc; p.G_tot = G_tot; p.S0 = S0; p.S_init = S_init; p.S_last = S_last;
    p.P = P; p.BH = BH; p.d_k = d_k; p.d_v = d_v; p.rows_per_block = d_k / K_blocks; p.groups = 1;
    return from_hip(zeco::launch_scan(p, static_cast<hipStream_t>(stream)));
}

// ---- two-level (tree of depth two) scan ----------------------------------------------------------------
size_t zeco_state_scan_tree_workspace(int32_t P, int32_t BH, int32_t d_k, int32_t d_v, int32_t gate_per_head) {
    if (P <= 0 || BH <= 0 || d_k <= 0 || d_v <= 0) return 0;
    return tree_floats(P, BH, d_k, d_v, gate_per_head) * sizeof(float);
}

zeco_status zeco_state_scan_tree(int32_t P, int32_t BH, int32_t d_k, int32_t d_v, const float *S_loc,
                                 const float *G_tot, const float *S0, float *S_init, float *S_last,
                                 int32_t direction, int32_t gate_per_head, void *workspace,
                                 size_t workspace_bytes, void *stream) {
    const int g = P > 0 ? tree_group(P) : 0;
    if (P <= 0 || g == P || BH <= 0)   // nothing to split (or an argument the plain scan reports)
        return zeco_state_scan(P, BH, d_k, d_v, d_k >= 16 && d_k % 16 == 0 ? 16 : 1, S_loc, G_tot, S0, S_init, S_last,
                               direction, gate_per_head, stream);
    if (d_k <= 0 || d_v <= 0 || d_k % 16 != 0) return ZECO_ERR_INVALID_ARG;
    if (direction != 0 && direction != 1) return ZECO_ERR_INVALID_ARG;
    if (gate_per_head != 0 && gate_per_head != 1) return ZECO_ERR_INVALID_ARG;
    if (!S_loc || !G_tot || !S_init) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(S_loc) || !aligned16(S_init) || !aligned16(S0) || !aligned16(S_last) ||
        (reinterpret_cast<uintptr_t>(G_tot) & 3u))
        return ZECO_ERR_INVALID_ARG;
    if ((int64_t)BH * 16 > (int64_t)1 << 30 || P / g > 65535) return ZECO_ERR_INVALID_ARG;
    if (d_v % 4 != 0) return ZECO_ERR_UNSUPPORTED;
    if (workspace_bytes < zeco_state_scan_tree_workspace(P, BH, d_k, d_v, gate_per_head)) return ZECO_ERR_WORKSPACE;
    if (!workspace || !aligned16(workspace)) return ZECO_ERR_INVALID_ARG;

    zeco::ScanParams p;
    p.reverse = direction; p.gate_per_head = gate_per_head;
    p.BH = BH; p.d_k = d_k; p.d_v = d_v; p.rows_per_block = d_k / 16;
    p.S_loc = S_loc; p.G_tot = G_tot; p.S0 = S0; p.S_init = S_init; p.S_last = S_last;
    p.P = P; p.groups = 1;
    return from_hip(launch_scan_tree(p, static_cast<float *>(workspace), static_cast<hipStream_t>(stream)));
}

size_t zeco_state_scan_tree_static_limit(void) { return kStaticScratchBytes; }

zeco_status zeco_state_scan_tree_static(int32_t P, int32_t BH, int32_t d_k, int32_t d_v, const float *S_loc,
                                        const float *G_tot, const float *S0, float *S_init, float *S_last,
                                        int32_t direction, int32_t gate_per_head, void *stream) {
    // the size check comes first: it needs nothing but the four sizes
    const size_t need = zeco_state_scan_tree_workspace(P, BH, d_k, d_v, gate_per_head);
    if (need > kStaticScratchBytes) return ZECO_ERR_SCRATCH_LIMIT;
    if (need == 0)   // the chain is not split (or an argument is bad, which the workspace variant reports)
        return zeco_state_scan_tree(P, BH, d_k, d_v, S_loc, G_tot, S0, S_init, S_last, direction, gate_per_head,
                                    nullptr, 0, stream);
    // Validate what zeco_state_scan_tree validates before the first HIP call (the lookup below is one).
    if (d_k % 16 != 0 || (direction != 0 && direction != 1) || (gate_per_head != 0 && gate_per_head != 1))
        return ZECO_ERR_INVALID_ARG;
    if (!S_loc || !G_tot || !S_init) return ZECO_ERR_INVALID_ARG;
    void *scratch = nullptr;
    if (static_scratch(&scratch) != hipSuccess) return ZECO_ERR_HIP;
    // The three passes write every byte of the scratch they later read (group end states and decay sums, then
    // the states entering the groups), so whatever an earlier call left there does not matter.
    return zeco_state_scan_tree(P, BH, d_k, d_v, S_loc, G_tot, S0, S_init, S_last, direction, gate_per_head,
                                scratch, kStaticScratchBytes, stream);
}

zeco_status zeco_apply_init_state(const zeco_gla_desc *d, const void *q, const float *G_cum,
                                  const float *S_init, void *o, int32_t flags, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !G_cum || !S_init || !o) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(G_cum) || !aligned16(S_init) || !aligned16(o))
        return ZECO_ERR_INVALID_ARG;
    if (flags & ~(ZECO_APPLY_FIRST_SEGMENT_ZERO | ZECO_APPLY_DENSE)) return ZECO_ERR_INVALID_ARG;

    zeco::ApplyParams p;
    fill_apply_params(p, d, d->P, d->L);
    p.q = q; p.G_cum = G_cum; p.S_init = S_init; p.o = o;
    p.p0 = (flags & ZECO_APPLY_FIRST_SEGMENT_ZERO) ? 1 : 0;
    p.dense = (flags & ZECO_APPLY_DENSE) ? 1 : 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (d->io_dtype == ZECO_F32) return from_hip(zeco::launch_apply_f32(p, d->d_k, d->d_v, s));
    if (p.dense) set_apply_share(p, d->L, 256, p.pad == 0);
    return from_hip(zeco::launch_apply_bf16(p, d->d_k, d->d_v, s));
}

// ---- segments of unequal length ---------------------------------------------------------------------------
static zeco_status check_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (T < (int64_t)d->P * d->C || T > (int64_t)1 << 40) return ZECO_ERR_INVALID_ARG;
    if (d->B == 0) return ZECO_OK;
    if (!seg_start || (reinterpret_cast<uintptr_t>(seg_start) & 7u)) return ZECO_ERR_INVALID_ARG;
    return ZECO_OK;
}

zeco_status zeco_gla_local_fwd_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T,
                                      const void *q, const void *k, const void *v, const void *g, void *o,
                                      float *S_loc, float *G_cum, float *G_tot, void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !o || !S_loc || !G_cum || !G_tot) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(o) ||
        !aligned16(S_loc) || !aligned16(G_cum) || !aligned16(G_tot))
        return ZECO_ERR_INVALID_ARG;
    static_assert(sizeof(long long) == sizeof(int64_t), "the kernels read the table as long long");
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.q = q; p.k = k; p.v = v; p.g = g; p.o = o;
    p.S_loc = S_loc; p.G_cum = G_cum; p.G_tot = G_tot;
    p.seg_start = reinterpret_cast<const long long *>(seg_start); p.T = T;
    hipStream_t s = static_cast<hipStream_t>(stream);
    return from_hip(launch_phase(p, d, 0, s));
}

zeco_status zeco_apply_init_state_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T,
                                         const void *q, const float *G_cum, const float *S_init, void *o,
                                         int32_t flags, void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !G_cum || !S_init || !o) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(G_cum) || !aligned16(S_init) || !aligned16(o))
        return ZECO_ERR_INVALID_ARG;
    if (flags & ~(ZECO_APPLY_FIRST_SEGMENT_ZERO | ZECO_APPLY_DENSE)) return ZECO_ERR_INVALID_ARG;
    zeco::ApplyParams p;
    fill_apply_params(p, d, d->P, d->L);
    p.dense = (flags & ZECO_APPLY_DENSE) ? 1 : 0;
    // a launch sized for the longest segment allowed; the lengths need not divide into the workgroups' shares
    set_apply_share(p, d->L, (p.dense && d->io_dtype == ZECO_BF16) ? 256 : 1024, false);
    p.q = q; p.G_cum = G_cum; p.S_init = S_init; p.o = o;
    p.seg_start = reinterpret_cast<const long long *>(seg_start); p.T = T;
    p.p0 = (flags & ZECO_APPLY_FIRST_SEGMENT_ZERO) ? 1 : 0;
    p.dense = (flags & ZECO_APPLY_DENSE) ? 1 : 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (d->io_dtype == ZECO_F32) return from_hip(zeco::launch_apply_f32(p, d->d_k, d->d_v, s));
    return from_hip(zeco::launch_apply_bf16(p, d->d_k, d->d_v, s));
}

// The two phases of Alg. 1's own schedule over the same table (bf16 only, like the equal-length calls).
zeco_status zeco_gla_local_state_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T,
                                        const void *k, const void *v, const void *g, float *S_loc,
                                        float *G_tot, void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!k || !v || !g || !S_loc || !G_tot) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(S_loc) || !aligned16(G_tot))
        return ZECO_ERR_INVALID_ARG;
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.k = k; p.v = v; p.g = g; p.S_loc = S_loc; p.G_tot = G_tot;
    p.seg_start = reinterpret_cast<const long long *>(seg_start); p.T = T;
    return from_hip(launch_phase(p, d, 1, static_cast<hipStream_t>(stream)));
}

zeco_status zeco_gla_fwd_from_state_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T,
                                           const void *q, const void *k, const void *v, const void *g,
                                           const float *S_init, void *o, void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !S_init || !o) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(S_init) || !aligned16(o))
        return ZECO_ERR_INVALID_ARG;
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.q = q; p.k = k; p.v = v; p.g = g; p.o = o; p.S_init = S_init;
    p.seg_start = reinterpret_cast<const long long *>(seg_start); p.T = T;
    return from_hip(launch_phase(p, d, 2, static_cast<hipStream_t>(stream)));
}

// The backward's building blocks over the same table (bf16 only, like the equal-length calls).
zeco_status zeco_gla_bwd_dstate_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T,
                                       const void *q, const void *g, const void *dO, float *dS_loc,
                                       void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !g || !dO || !dS_loc) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(g) || !aligned16(dO) || !aligned16(dS_loc)) return ZECO_ERR_INVALID_ARG;
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.k = q; p.v = dO; p.g = g; p.S_loc = dS_loc; p.kscale = d->scale;
    p.seg_start = reinterpret_cast<const long long *>(seg_start); p.T = T;
    return from_hip(launch_phase(p, d, 3, static_cast<hipStream_t>(stream)));
}

zeco_status zeco_gla_bwd_from_state_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T,
                                           const void *q, const void *k, const void *v, const void *g,
                                           const void *dO, const float *S_init, const float *S_last,
                                           const float *dS_in, void *dq, void *dk, void *dv, float *dg,
                                           void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    const size_t need = zeco_gla_bwd_from_state_workspace(d);   // sized for the bound on the lengths
    if (workspace_bytes < need) return ZECO_ERR_WORKSPACE;
    if (need && (!workspace || !aligned16(workspace))) return ZECO_ERR_INVALID_ARG;
    if (!q || !k || !v || !g || !dO || !S_init || !S_last || !dS_in || !dq || !dk || !dv || !dg)
        return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(dO) ||
        !aligned16(S_init) || !aligned16(S_last) || !aligned16(dS_in) || !aligned16(dq) || !aligned16(dk) ||
        !aligned16(dv) || !aligned16(dg))
        return ZECO_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    float *S_ck = need ? static_cast<float *>(workspace) : nullptr;
    const zeco_status sq = bwd_dq_pass(d, d->P, d->L, q, k, v, g, dO, S_init, S_last, dq, dg, nullptr, nullptr, S_ck, s,
                                       seg_start, T);
    if (sq != ZECO_OK) return sq;
    return bwd_dv_dk_passes(d, d->P, d->L, q, k, v, g, dO, S_init, S_last, dS_in, dk, dv, dg, S_ck, s, seg_start, T);
}

// The whole forward and the whole backward over the same table, each in one call: the phases of Alg. 1 (states,
// scan, output pass) and of the backward (forward states and their scan, dQ pass with the segments' state
// gradients, reverse scan, dV and dK passes).
//
// Segments of up to 33 chunks are worked on as given, so that the call repeats the separate calls over the table bit for
// bit; that is what the bound is for, and not that a cut would not pay.  Longer ones are cut: the segments together are
// one run of tokens, whose pieces need not end where they do, so the run is cut as in zeco_gla_fused_fwd, on the device
// (launch_plan), where the table is.  Forward and backward, d = 128, segments of up to 2112 (whole) / 2113 (cut) tokens: 16
// segments, 1 head 628 / 170 us, 4 heads 626 / 345 us, 16 heads 1044 / 1069 us; 3 segments, 16 heads 631 / 274 us.  8 segments of
// 1160 .. 9287 tokens, 16 heads: 3.15 ms as given (the longest segment's chain), 1.02 ms in 16 pieces.
constexpr int kWholeSegments = 33 * 64;
struct VarlenLayout {   // workspace carve-up, in floats
    int slots;          // pieces, or segments
    size_t state, off_Sinit, off_Gtot, off_dSloc, off_dSin, off_ck, off_table, total;
};
static VarlenLayout varlen_layout(const zeco_gla_desc *d, bool backward) {
    VarlenLayout w;
    const bool cut = d->L > kWholeSegments;
    const long long T = (long long)d->P * d->L;         // no valid table covers more
    const long long n = cut ? pieces_for(d, T, false, false) : 0;
    w.slots = n > d->P ? (int)n : d->P;
    const size_t slots = (size_t)w.slots * d->B * d->H, bh = (size_t)d->B * d->H;
    w.state = (size_t)d->d_k * d->d_v;
    w.off_Sinit = slots * w.state;                      // S_loc [slots] first
    w.off_Gtot = w.off_Sinit + (slots + bh) * w.state;  // S_init [slots] and one more: the final state
    w.off_dSloc = w.off_Gtot + ((slots * (d->g_per_head ? 1 : d->d_k) + 3) & ~(size_t)3);
    w.off_dSin = w.off_ck = w.off_table = w.off_dSloc;
    if (backward) {
        w.off_dSin = w.off_dSloc + slots * w.state;
        w.off_ck = w.off_dSin + slots * w.state;
        // checkpoints: of the segments, or of n pieces, (whole chunks of a piece) / 8 each at most
        const size_t per = cut ? (size_t)T / 512 : (size_t)d->P * bwd_checkpoints(d->L);
        w.off_table = w.off_ck + per * bh * w.state;
    }
    w.total = w.off_table + (cut ? 2 * ((size_t)w.slots + 4) : 0);
    return w;
}

size_t zeco_gla_fused_fwd_varlen_workspace(const zeco_gla_desc *desc) {
    if (check_desc(desc, true) != ZECO_OK) return 0;
    return varlen_layout(desc, false).total * sizeof(float);
}
size_t zeco_gla_fused_bwd_varlen_workspace(const zeco_gla_desc *desc) {
    if (check_desc(desc, true) != ZECO_OK) return 0;
    return varlen_layout(desc, true).total * sizeof(float);
}

// What the passes of a varlen call work on: the caller's table, or a table of pieces made from it (enqueued here).
struct VarlenRun {
    int P = 0, L = 0, plan = 0;
    const int64_t *table = nullptr;
    const long long *used = nullptr;
};
static hipError_t varlen_run(VarlenRun &r, const zeco_gla_desc *d, const VarlenLayout &w, float *ws, const int64_t *seg_start,
                             int64_t T, hipStream_t s) {
    r.P = d->P; r.L = d->L; r.table = seg_start;
    if (d->L <= kWholeSegments) return hipSuccess;
    const long long run = (long long)d->P * d->L < T ? (long long)d->P * d->L : T;
    long long n = pieces_for(d, run, false, false);
    if (n > w.slots) n = w.slots;
    zeco::SegPlan p;
    p.seg_start = reinterpret_cast<const long long *>(seg_start);
    p.table = reinterpret_cast<long long *>(ws + w.off_table);
    p.P = d->P; p.slots = w.slots; p.n = (int)n; p.L = d->L; p.T = T;
    p.ck_even = bwd_checkpoints(longest_tokens(cut_of(run, n)));
    p.ck_segments = bwd_checkpoints(d->L);
    r.P = r.plan = w.slots; r.table = reinterpret_cast<const int64_t *>(p.table); r.used = p.table + w.slots + 1;
    return zeco::launch_plan(p, s);
}

zeco_status zeco_gla_fused_fwd_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T, const void *q,
                                      const void *k, const void *v, const void *g, const float *S0, void *o,
                                      float *S_last, void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !o || !workspace) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(o) || !aligned16(S0) ||
        !aligned16(S_last) || !aligned16(workspace))
        return ZECO_ERR_INVALID_ARG;
    const VarlenLayout w = varlen_layout(d, false);
    if (workspace_bytes < w.total * sizeof(float)) return ZECO_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    float *Sloc = static_cast<float *>(workspace), *Sinit = Sloc + w.off_Sinit, *Gtot = Sloc + w.off_Gtot;
    VarlenRun run;
    if (varlen_run(run, d, w, Sloc, seg_start, T, s) != hipSuccess) return ZECO_ERR_HIP;
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.P = run.P; p.plan = run.plan;
    p.seg_start = reinterpret_cast<const long long *>(run.table); p.T = T;
    p.k = k; p.v = v; p.g = g; p.S_loc = Sloc; p.G_tot = Gtot;
    if (launch_phase(p, d, 1, s) != hipSuccess) return ZECO_ERR_HIP;
    zeco::ScanParams sp;
    sp.S_loc = Sloc; sp.G_tot = Gtot; sp.S0 = S0; sp.S_init = Sinit; sp.S_last = S_last;
    sp.P = run.P; sp.P_used = run.used; sp.groups = 1; sp.BH = d->B * d->H; sp.d_k = d->d_k; sp.d_v = d->d_v;
    sp.rows_per_block = d->d_k / 16; sp.gate_per_head = d->g_per_head;
    if (zeco::launch_scan(sp, s) != hipSuccess) return ZECO_ERR_HIP;
    p.q = q; p.o = o; p.S_init = Sinit; p.S_loc = nullptr; p.G_tot = nullptr;
    return from_hip(launch_phase(p, d, 2, s));
}

zeco_status zeco_gla_fused_bwd_varlen(const zeco_gla_desc *d, const int64_t *seg_start, int64_t T, const void *q,
                                      const void *k, const void *v, const void *g, const void *dO,
                                      const float *S0, const float *dS_T, void *dq, void *dk, void *dv, float *dg,
                                      float *dS0, void *workspace, size_t workspace_bytes, void *stream) {
    const zeco_status st = check_varlen(d, seg_start, T);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !dO || !dq || !dk || !dv || !dg || !workspace) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(dO) || !aligned16(S0) ||
        !aligned16(dS_T) || !aligned16(dq) || !aligned16(dk) || !aligned16(dv) || !aligned16(dg) || !aligned16(dS0) ||
        !aligned16(workspace))
        return ZECO_ERR_INVALID_ARG;
    const VarlenLayout w = varlen_layout(d, true);
    if (workspace_bytes < w.total * sizeof(float)) return ZECO_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t slots = (size_t)w.slots * d->B * d->H;
    float *ws = static_cast<float *>(workspace);
    float *Sloc = ws, *Sinit = ws + w.off_Sinit, *Slast = Sinit + slots * w.state, *Gtot = ws + w.off_Gtot;
    float *dSloc = ws + w.off_dSloc, *dSin = ws + w.off_dSin;
    float *S_ck = bwd_checkpoints(d->L) > 0 ? ws + w.off_ck : nullptr;
    VarlenRun run;
    if (varlen_run(run, d, w, ws, seg_start, T, s) != hipSuccess) return ZECO_ERR_HIP;
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.P = run.P; p.plan = run.plan;
    p.seg_start = reinterpret_cast<const long long *>(run.table); p.T = T;
    p.k = k; p.v = v; p.g = g; p.S_loc = Sloc; p.G_tot = Gtot;
    if (launch_phase(p, d, 1, s) != hipSuccess) return ZECO_ERR_HIP;
    zeco::ScanParams sp;
    sp.S_loc = Sloc; sp.G_tot = Gtot; sp.S0 = S0; sp.S_init = Sinit; sp.S_last = Slast;
    sp.P = run.P; sp.P_used = run.used; sp.groups = 1; sp.BH = d->B * d->H; sp.d_k = d->d_k; sp.d_v = d->d_v;
    sp.rows_per_block = d->d_k / 16; sp.gate_per_head = d->g_per_head;
    if (zeco::launch_scan(sp, s) != hipSuccess) return ZECO_ERR_HIP;
    zeco_status zs = bwd_dq_pass(d, run.P, run.L, q, k, v, g, dO, Sinit, Slast, dq, dg, dSloc, nullptr, S_ck, s, run.table, T,
                                 nullptr, run.plan);
    if (zs != ZECO_OK) return zs;
    sp.S_loc = dSloc; sp.S0 = dS_T; sp.S_init = dSin; sp.S_last = dS0; sp.reverse = 1;
    if (zeco::launch_scan(sp, s) != hipSuccess) return ZECO_ERR_HIP;
    return bwd_dv_dk_passes(d, run.P, run.L, q, k, v, g, dO, Sinit, Slast, dSin, dk, dv, dg, S_ck, s, run.table, T, nullptr,
                            run.plan);
}

// ---- chunk-decay form of the local pass and the correction ---------------------------------------------
zeco_status zeco_gla_local_fwd_chunk_decay(const zeco_gla_desc *d, const void *q, const void *k,
                                           const void *v, const void *g, void *o, float *S_loc,
                                           float *G_chunk, float *G_tot, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !k || !v || !g || !o || !S_loc || !G_chunk || !G_tot) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(g) || !aligned16(o) ||
        !aligned16(S_loc) || !aligned16(G_chunk) || !aligned16(G_tot))
        return ZECO_ERR_INVALID_ARG;
    if (d->io_dtype != ZECO_BF16 || d->g_per_head) return ZECO_ERR_UNSUPPORTED;
    zeco::ChunkParams p;
    fill_chunk_params(p, d);
    p.q = q; p.k = k; p.v = v; p.g = g; p.o = o; p.S_loc = S_loc; p.G_tot = G_tot; p.G_chunk = G_chunk;
    return from_hip(zeco::launch_chunk_bf16(p, d->d_k, d->d_v, chunk_gate(d), 6,
                                            static_cast<hipStream_t>(stream)));
}

zeco_status zeco_apply_init_state_chunk_decay(const zeco_gla_desc *d, const void *q, const void *g,
                                              const float *G_chunk, const float *S_init, void *o,
                                              int32_t flags, void *stream) {
    const zeco_status st = check_desc(d, true);
    if (st != ZECO_OK) return st;
    if (d->B == 0) return ZECO_OK;   // empty batch: nothing to do
    if (!q || !g || !G_chunk || !S_init || !o) return ZECO_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(g) || !aligned16(G_chunk) || !aligned16(S_init) || !aligned16(o))
        return ZECO_ERR_INVALID_ARG;
    if (flags & ~(ZECO_APPLY_FIRST_SEGMENT_ZERO | ZECO_APPLY_DENSE)) return ZECO_ERR_INVALID_ARG;
    if (d->io_dtype != ZECO_BF16 || d->g_per_head) return ZECO_ERR_UNSUPPORTED;
    zeco::ApplyParams p;
    fill_apply_params(p, d, d->P, d->L);
    p.q = q; p.g = g; p.g_bf16 = d->g_dtype == ZECO_BF16; p.G_chunk = G_chunk; p.S_init = S_init; p.o = o;
    p.p0 = (flags & ZECO_APPLY_FIRST_SEGMENT_ZERO) ? 1 : 0;
    p.dense = (flags & ZECO_APPLY_DENSE) ? 1 : 0;
    return from_hip(zeco::launch_apply_cd_bf16(p, d->d_k, d->d_v, static_cast<hipStream_t>(stream)));
}

zeco_status zeco_hbm_copy(void *dst, const void *src, size_t bytes, void *stream) {
    if (!dst || !src || !aligned16(dst) || !aligned16(src) || bytes % 16 != 0) return ZECO_ERR_INVALID_ARG;
    return from_hip(zeco::launch_copy(dst, src, bytes, static_cast<hipStream_t>(stream)));
}

zeco_status zeco_hbm_mix(void *dst, const void *src, size_t slice_bytes, int32_t reads, int32_t writes, void *stream) {
    if (!dst || !src || !aligned16(dst) || !aligned16(src) || slice_bytes % 16 != 0) return ZECO_ERR_INVALID_ARG;
    const int ok[][2] = {{1, 0}, {0, 1}, {1, 1}, {2, 1}, {3, 1}, {4, 1}, {5, 3}, {3, 2}};
    bool found = false;
    for (auto &m : ok) found = found || (m[0] == reads && m[1] == writes);
    if (!found) return ZECO_ERR_UNSUPPORTED;
    return from_hip(zeco::launch_mix(dst, src, slice_bytes, reads, writes, static_cast<hipStream_t>(stream)));
}

const char *zeco_status_string(int32_t status) {
    switch (status) {
        case ZECO_OK: return "ok";
        case ZECO_ERR_INVALID_ARG: return "invalid argument";
        case ZECO_ERR_UNSUPPORTED: return "unsupported configuration";
        case ZECO_ERR_WORKSPACE: return "workspace too small";
        case ZECO_ERR_HIP: return "HIP runtime error";
        case ZECO_ERR_SCRATCH_LIMIT: return "problem needs more than the library's static scratch";
        default: return "unknown status";
    }
}

int32_t zeco_version(void) { return 100; }

}  // extern "C"
