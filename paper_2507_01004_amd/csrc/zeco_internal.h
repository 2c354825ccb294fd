// Host-side launcher interface between the C ABI (zeco_api.hip) and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace zeco {

// Gate layouts: kGateF32 / kGateBF16 = one log decay per (token, head, channel); kGateHead = one fp32
// log decay per (token, head), shared by all channels (g, G_cum [B,T,H] contiguous; G_tot [P,B,H]).
enum GateMode { kGateF32 = 0, kGateBF16 = 1, kGateHead = 2 };
// added to the gate layout handed to launch_chunk_bf16: decay factors of the tiles counted from half the chunk's
// total log decay (twice the range of gates, one more multiplication of the state per chunk)
constexpr int kGateWide = 4;

// Cut of a run of `len` tokens into n pieces of whole 64-token chunks, as even as that allows: the last `rem` pieces
// hold base + 1 chunks, the others base (base >= 1), and the first one the len % 64 tokens left over as well, so
// that no piece is shorter than 64 tokens whatever the length, and all pieces begin where a forward pass over the
// whole run, which makes its first chunk the short one, begins a chunk.  n = 0: no cut, the launch's segments are
// used as they are.  With a cut the launch's "segments" are pieces: piece s is piece s % n of run s / n.
struct Cut {
    int n = 0, base = 0, rem = 0;
    long long len = 0;
};

// Table of pieces in the segments' place, made on the device from the caller's table of segments (which the host
// cannot read): table [slots + 4] int64 = piece offsets [slots + 1], pieces in use, upper bound of their lengths,
// checkpoints per piece.  The launches have a workgroup per slot; those of unused slots leave.
// When all P segments keep the rules they are one run of tokens and it is cut into n even pieces (as Cut does); with a
// segment that breaks them the pieces are the segments, under the caller's bound, and the kernels skip that one.
struct SegPlan {
    const long long *seg_start;
    long long *table;
    int P, slots, n;
    long long L, T;              // bound on the segments' lengths, tokens per batch entry
    int ck_even, ck_segments;    // checkpoints per piece in the two cases
};

struct ChunkParams {
    int B, P, H, L;
    int n_chunks;              // ceil(L / 64)
    int pad = 0;               // 64 n_chunks - L: the first chunk processed holds 64 - pad tokens
    int plan = 0;              // slots of a table written by launch_plan (SegPlan); 0: seg_start is the caller's own table
    float scale;
    Cut cut;                   // P counts pieces, n_chunks is the longest piece's (the stride of G_chunk), L and pad are unused
    // Segments of unequal length (modes 0 to 3 of the bf16 kernel, and the fp32 kernel): segment p covers tokens
    // [seg_start[p], seg_start[p+1]) of the T tokens of every batch entry; L is then the upper bound of the
    // lengths, n_chunks and pad are unused.
    const long long *seg_start = nullptr;
    long long T = 0;           // tokens per batch entry, in every launch
    long long sb, st, sh;      // q/k/g element strides
    long long vb, vt, vh;      // v/o element strides
    const void *q, *k, *v, *g;
    void *o;
    float *S_loc, *G_cum, *G_tot;
    const float *S_init;       // [P,B,H,d_k,d_v] initial states (modes that start from a given state)
    const float *G_off = nullptr;   // [P,B,H,d_k] ([P,B,H] per-head) log decay preceding each segment, as pairs (mode 5 only)
    float *G_chunk = nullptr;       // [B,P,n_chunks,H,d_k] log decay from the segment start to each chunk's start (mode 6 only)
    // Output pass over a run in one piece (mode 7), for a training step: the states entering the pieces of `emit` (a cut of the same run),
    // S_emit [emit.n, B, H, d_k, d_v], for a backward on those pieces; and the end state a second time, S_loc2
    float *S_emit = nullptr, *S_loc2 = nullptr;
    Cut emit;
    // 1: G_tot as pairs (mode 1) - every log decay with what fp32 leaves off it beside it, [.., 2], so that sums of log
    // decays run on across the pieces of a segment as precisely as inside one
    int pairs = 0;
    int local = 0;             // 1: one of the passes of a cut local pass (fp32 kernels: log decays are summed as in the local pass)
    // mode 1: n > 0 may leave out every n-th segment (the last piece of each of the caller's segments, cut into n), whose end state
    // nobody reads
    int skip_last = 0;
    float kscale;              // backward modes: multiplier carried by the operand in the k role
};

struct ApplyParams {
    const void *q;
    const float *G_cum = nullptr;    // [B,T,H,d_k] per-token cumulative log decay, or
    const float *G_chunk = nullptr;  // [B,P,n_chunks,H,d_k] per-chunk one, together with
    const void *g = nullptr;         //   the log decays themselves (layout of q)
    int g_bf16 = 0;                  //   stored as bf16 (1) or fp32 (0)
    const float *S_init;
    void *o;
    int B, P, H, L;
    int p0;                    // first segment to correct
    int seg_step = 1;          // ... and every seg_step-th one after it
    int tokens_per_wg;         // multiple of 64
    int n_chunks, pad;         // 64-token blocks per segment, ceil(L / 64), and 64 n_chunks - L: the first block is the short one
    int wgs_per_seg;           // workgroups per segment, ceil(64 n_chunks / tokens_per_wg)
    const long long *seg_start = nullptr;   // segments of unequal length (the kernels that read G_cum):
    long long T = 0;                        //   as in ChunkParams; n_chunks, pad, wgs_per_seg describe the bound L
    Cut cut;                   // as in ChunkParams; wgs_per_seg describes the longest piece
    int gate_per_head = 0;     // 1: G_cum [B,T,H] (bf16 kernel only)
    int dense = 0;             // 1: stream every token, also where exp(G_cum) has vanished
    float scale;
    long long sb, st, sh, vb, vt, vh;
};

// `groups` independent chains of P segments each: S_loc, S_init [groups*P, BH, d_k, d_v],
// G_tot [groups*P, BH, d_k], S0 and S_last [groups, BH, d_k, d_v].
struct ScanParams {
    const float *S_loc, *G_tot, *S0;
    float *S_init, *S_last;      // either may be null (not stored)
    float *S_last2 = nullptr;    // optional: the end states a second time
    int P, BH, d_k, d_v, rows_per_block, groups;
    const long long *P_used = nullptr;   // optional, one chain only: its length, on the device (at most P)
    int reverse = 0;             // 1: chain runs from segment P-1 down to 0
    // optional, each on its own: G_pre [groups*P, BH, d_k] = sum of G_tot over the earlier segments of the
    // chain (forward chains only), G_sum [groups, BH, d_k] = sum over all of them ([.., BH] with one decay per head)
    float *G_pre = nullptr, *G_sum = nullptr;
    int pairs = 0;               // 1: G_tot and G_pre as pairs (see ChunkParams), added up in 64 bits
    int gate_per_head = 0;       // 1: G_tot [groups*P, BH], one log decay per head
};

// dQ pass; dK, dV and dG pass (gla_bwd_qk.hip).  x, y: [B,T,H,d_v] operands (strides vb, vt, vh); z, z2, g, out:
// [B,T,H,d_k] (strides sb, st, sh); W_init [P,B,H,d_k,d_v] fp32; dg [B,T,H,d_k] fp32 contiguous (the dQ
// pass leaves q .* dq there, the dK pass turns it into dG); S_init, S_last: forward states (dK pass).
// With per-head gates g and dg are [B,T,H] and the channel sums are taken before anything is stored.
struct BwdQKParams {
    int B, P, H, L, n_chunks;    // n_chunks = ceil(L / 64)
    int pad = 0;                 // 64 n_chunks - L: the first chunk processed holds 64 - pad tokens
    int plan = 0;                // as in ChunkParams
    int n_ck = 0;
    Cut cut;                     // as in ChunkParams
    const long long *seg_start = nullptr;   // segments of unequal length, as in ChunkParams (L = bound on the
    long long T = 0;                        //   lengths, T = tokens per batch entry)
    long long sb, st, sh, vb, vt, vh;
    const void *x, *y, *z, *z2, *g;
    void *out;
    void *out2 = nullptr;        // dK pass: dv, [B,T,H,d_v] (strides vb, vt, vh)
    float *dg;
    const float *W_init, *S_init, *S_last;
    float zscale, oscale;        // multipliers of the gated operand and of the output
    // dQ pass only, optional: also emit each segment's state gradient from dS = 0,
    // dS_loc [P,B,H,d_k,d_v] = qscale * sum_t (q_t .* exp(G_t))^T x_t, and its total log decay G_tot_out
    float *dS_loc = nullptr, *G_tot_out = nullptr;
    float qscale = 1.f;
    // optional checkpoints that re-anchor dG: S_ck [B*P*H, n_ck, d_k, d_v], the forward state entering every
    // 8th chunk (chunks 8, 16, ..) of each segment; written by the dQ pass, read by the dK pass.  With it the dQ
    // pass must be launched with short_last = 1 (the short chunk of a ragged length at the segment's end).
    int short_last = 0;
    float *S_ck = nullptr;
};

// A kernel that uses more dynamic LDS than the default limit has the limit raised once per device (the
// attribute belongs to the function on that device), not at every launch.  One static object per kernel
// instantiation; devices beyond the 64 the mask covers are simply set every time.
struct LdsLimit {
    std::atomic<unsigned long long> done{0};
    hipError_t raise(const void *kernel, int bytes) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const unsigned long long bit = (dev >= 0 && dev < 64) ? 1ull << dev : 0ull;
        if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
        return e;
    }
};

// Each returns hipSuccess or the launch error.  d_k, d_v in {64,128}.
// fp32 kernels: chunk length C in {16, 32, 64}; mode 0 local pass, 1 states only, 2 output pass from S_init, 3 backward state pass, 4 dV
// pass, 5 (as in the bf16 kernel below).  p.n_chunks and p.pad count chunks of f32_chunk tokens, the length the kernel of that mode
// works in.
int f32_chunk(const ChunkParams &p, int C, int mode);
hipError_t launch_chunk_f32(const ChunkParams &p, int d_k, int d_v, int C, int mode, hipStream_t s);
// mode: 0 local pass (o, S_loc, G_cum, G_tot), 1 states only (S_loc, G_tot), 2 output pass from S_init (o),
// 3 backward state pass (k := q, v := dO; S_loc := dS leaving the segment), 5 output pass from S_init that also
// writes G_cum counted from G_off (o, G_cum), 6 local pass with the cumulative decay
// per chunk instead of per token (o, S_loc, G_chunk, G_tot; per-channel gates only), 7 mode 2 over whole runs:
// S_init may be null (zero), also the end states (S_loc) and, for a backward, S_emit and S_loc2, each if given
hipError_t launch_chunk_bf16(const ChunkParams &p, int d_k, int d_v, int gate_mode, int mode, hipStream_t s);
hipError_t launch_apply_f32(const ApplyParams &p, int d_k, int d_v, hipStream_t s);
hipError_t launch_apply_bf16(const ApplyParams &p, int d_k, int d_v, hipStream_t s);
// from (g, G_chunk) instead of G_cum; per-channel gates
hipError_t launch_apply_cd_bf16(const ApplyParams &p, int d_k, int d_v, hipStream_t s);
hipError_t launch_scan(const ScanParams &p, hipStream_t s);
hipError_t launch_plan(const SegPlan &p, hipStream_t s);
// reverse = false: dQ (x = dO, y = v, z = k, z2 = q, W_init = forward states); true: dK (x = v, y = dO,
// z = q, z2 = k, W_init = state gradients, out2 = dv; must run after the dQ pass, whose q .* dq it consumes)
hipError_t launch_bwd_qk(const BwdQKParams &p, int d_k, int d_v, int gate_mode, bool reverse, hipStream_t s);
// the same two passes on fp32 tensors (gla_bwd_f32.hip), chunk length C in {16, 32, 64}; no by-products
hipError_t launch_bwd_qk_f32(const BwdQKParams &p, int d_k, int d_v, int C, bool reverse, hipStream_t s);
// per-head log decays: G_cum [B,T,H] += G_pre [T/len, B, H] of the piece each token lies in
hipError_t launch_gate_offset_head(float *G_cum, const float *G_pre, int B, long long T, int H, int len, hipStream_t s);
hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s);
// reads x writes 16-byte streams over slices of slice_bytes each (calibration of the HBM rate of a traffic mix)
hipError_t launch_mix(void *dst, const void *src, size_t slice_bytes, int reads, int writes, hipStream_t s);

}  // namespace zeco
