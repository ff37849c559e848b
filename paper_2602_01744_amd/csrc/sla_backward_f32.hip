// Backward pass of sla_forward for the RetNet and GLA recurrences (Sec. 5.1) with SLA's head gates (Eq. 4-6), fp32
// tensors: every product in fp32 vector arithmetic, token by token, so that the gradients agree with an fp64
// evaluation to fp32 rounding.  (bf16 tensors take the block form on the matrix cores in sla_backward.hip.)
//
// Forward step, per head:  S_t = diag(alpha_t) S_{t-1} + G^K_t k_t^T v_t,  out_t = G^Q_t q_t S_t,  alpha_t =
// exp(log_decay_t) (GLA: one factor per key dimension and token; RetNet: one constant per head).  With X_t the
// gradient with respect to S_t including token t's own read-out term:
//     X_t = diag(alpha_{t+1}) X_{t+1} + q_t^T (G^Q_t dout_t)
//     dv_t = G^K_t k_t X_t         dG^K_t = v_t . (k_t X_t)
//     dk_t = G^K_t v_t X_t^T       dq_t = G^Q_t dout_t S_t^T       dG^Q_t = q_t . (dout_t S_t^T)
//     dlog_decay_t = rowsum(X_T' * S_T) + sum_{s >= t} (q_s * dq_s - k_s * dk_s)     (GLA; X_T' the caller's cotangent
//     of the final state; a writer j and a reader s contribute the same amount to q_s dq_s and to k_j dk_j and cross
//     token t's decay exactly when j < t <= s).  Where a row runs in segments, each is a sequence of its own: S_T and X_T'
//     are its exit state and the cotangent of that, so the sum restarts at every segment's end from an fp32 row sum.  It
//     is the shorter sum that decides: against 64 bits dlog_decay is off by 0.25 to 0.95 of what one pass leaves (T=130
//     64 x 64 4.7e-7 -> 2.6e-7, T=300 128 x 256 8.7e-7 -> 3.4e-7, T=4136 128 x 128 3.0e-6 -> 4.0e-7, 2-norms).
// Every output contracts a state over one of its two dimensions, so the pass is three sweeps that each carry one
// state tile in registers, sliced over the dimension that is not contracted:
//   dv sweep, backward in time, X[dk rows, 64 value columns]:  dv, partial dG^K, d_initial_state;
//   dq sweep, forward in time, S^T[dv rows, 64 key columns]:   dq, partial dG^Q, rowsum(X_T' * S_T);
//   dk sweep, backward in time, X^T[dv rows, 64 key columns]:  dk, dlog_decay (a running sum in fp64 per key column,
//                                                              over the sequence or the segment).
// The gate gradients then go through the head softmax in sla_bwd_logits_kernel (sla_backward.hip).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "sla.h"
#include "sla_gate_grad.h"
#include "sla_token_sweep.h"

namespace sla {

int launch_bwd_gates(const float* ql, const float* kl, float* gq, float* gk, size_t rows, int H, hipStream_t stream);
namespace {

using namespace tok;

struct FArgs {
    const float* q;        // [B,T,H,dk] (head-major: [B,H,T,dk])
    const float* k;
    const float* v;        // [B,T,H,dv]
    const float* dout;
    const float* ld;       // GLA: log-decay, laid out like q; else null
    const float* ld_head;  // RetNet: [H]; else null
    const float* gq;       // gates [B,T,H]
    const float* gk;
    const float* s0;       // [B,H,dk,dv] or null
    const float* dsf;
    float* dq;
    float* dk;
    float* dv;
    float* dld;            // GLA: laid out like q
    float* ds0;
    float* part_q;         // [dk/8][plane]: partial q . (dout S^T)
    float* part_k;         // [dv/8][plane]: partial v . (k X)
    float* corr;           // GLA: [B,H,dk] rowsum(X_T' * S_T)
    size_t plane;          // floats between partial planes (>= rows * H)
    size_t rows;           // tokens in all
    const int* cu;         // packed batch (see Where), else null
    int B, T, H;           // B: sequences; with nseg > 1 segments, nseg of them to a batch row of T tokens
    int nseg, seg_len;
    bool head_major;
};

// What a workgroup owns: a sequence, or with nseg > 1 one segment of seg_len tokens of a batch row, which then runs as
// a sequence of its own (me.b and me.bh number the segments, and with them the states).
__device__ __forceinline__ Where where_segment(const FArgs& a, int nslices, int block, int grid) {
    Where me = where(a, nslices, block, grid);
    if (a.nseg > 1 && me.bh >= 0) {
        const int t0 = (me.b % a.nseg) * a.seg_len;
        me.T = min(a.seg_len, a.T - t0);
        me.tok0 = (size_t)(me.b / a.nseg) * a.T + t0;
    }
    return me;
}

constexpr int kSc = 4;  // per-token scalars {G^Q, G^K, alpha of the head (RetNet; 1 for GLA), -}

// Where a head's rows start and how far tokens are apart, for a tensor of row width D.
struct Rows {
    size_t base, step;
};
__device__ __forceinline__ Rows rows_of(const FArgs& a, const Where& me, int D) {
    if (a.head_major)
        return Rows{((size_t)((me.b / a.nseg) * a.H + me.h) * a.T + (size_t)(me.b % a.nseg) * a.seg_len) * D, (size_t)D};
    return Rows{(me.tok0 * a.H + me.h) * D, (size_t)a.H * D};
}

// The decay factors of 16 tokens: staged like any fp32 tensor, written as exp(x); a token past the end gets 1.
template <int NC>
struct RegsA : RegsF<NC> {
    typedef RegsF<NC> Base;
    __device__ __forceinline__ f4 factor(int n, bool ok) const {
        const f4 x = this->x[n];
        return ok ? f4{__builtin_amdgcn_exp2f(x[0] * kLog2e), __builtin_amdgcn_exp2f(x[1] * kLog2e),
                       __builtin_amdgcn_exp2f(x[2] * kLog2e), __builtin_amdgcn_exp2f(x[3] * kLog2e)}
                  : f4{1.f, 1.f, 1.f, 1.f};
    }
    __device__ __forceinline__ void put_exp(float* dst, int t0, int T, int lt) const {
#pragma unroll
        for (int n = 0; n < Base::N; ++n) {
            const int it = lt + kLoaders * n, tok = it / (NC / 4), c4 = it % (NC / 4);
            if (it < Base::items) *(f4*)(dst + tok * NC + 4 * c4) = factor(n, t0 + tok < T);
        }
    }
    __device__ __forceinline__ void put_rows_exp(float* dst, int t0, int T, int lt) const {
#pragma unroll
        for (int n = 0; n < Base::N; ++n) {
            const int it = lt + kLoaders * n, tok = it / (NC / 4), c4 = it % (NC / 4);
            if (it < Base::items) *(f4*)(dst + tok * NC + row_slot<NC / 16>(4 * c4)) = factor(n, t0 + tok < T);
        }
    }
};

struct RegsG {  // the gates of 16 tokens (lanes 0..15 of the first loader wave)
    float gq, gk;
    __device__ __forceinline__ void load(const FArgs& a, size_t tok0, int h, int t0, int T, int lt) {
        const size_t i = (tok0 + (size_t)min(t0 + (lt & (kChunk - 1)), T - 1)) * a.H + h;
        gq = a.gq[i]; gk = a.gk[i];
    }
    __device__ __forceinline__ void put(float* dst, float head_alpha, int t0, int T, int lt) const {
        if (lt < kChunk) {
            const bool ok = t0 + lt < T;
            *(f4*)(dst + kSc * lt) = ok ? f4{gq, gk, head_alpha, 0.f} : f4{0.f, 0.f, 1.f, 0.f};
        }
    }
};

__device__ __forceinline__ float head_alpha_of(const FArgs& a, int h) {
    return a.ld_head ? __builtin_amdgcn_exp2f(a.ld_head[h] * kLog2e) : 1.f;
}

// ------------------------------------------------------------------------------------------------------------
// dv sweep: backward in time, X[dk rows, value columns].
// ------------------------------------------------------------------------------------------------------------
template <bool GLA, int DK, int DV>
__device__ __forceinline__ void dv_sweep(const FArgs& a, unsigned char* smem, int block, int grid) {
    constexpr int RT = DK / 16;
    constexpr int oK = 0, oQ = oK + kChunk * DK, oA = oQ + kChunk * DK, oV = oA + (GLA ? kChunk * DK : 0),
                  oDO = oV + kChunk * kSlice, oSC = oDO + kChunk * kSlice, kBuf = oSC + kSc * kChunk;
    float* lds = (float*)smem;
    const Where me = where_segment(a, DV / kSlice, block, grid);
    if (me.bh < 0) return;
    const int T = me.T, nch = (T + kChunk - 1) / kChunk;
    const Rows rk = rows_of(a, me, DK), rv = rows_of(a, me, DV);
    if (me.wave >= kWaves) {  // step c of the sweep covers tokens (nch - 1 - c) * 16 ...
        const int lt = me.tid - 64 * kWaves;
        const float ha = head_alpha_of(a, me.h);
        for (int c = 0; c <= nch; ++c) {
            if (c < nch) {
                const int t0 = (nch - 1 - c) * kChunk;
                float* buf = lds + (c & 1) * kBuf;
                RegsF<DK> xk, xq;
                RegsA<DK> xa;
                RegsF<kSlice> xv, xd;
                RegsG xs;
                xk.load(a.k + rk.base, rk.step, t0, T, lt); xq.load(a.q + rk.base, rk.step, t0, T, lt);
                if constexpr (GLA) xa.load(a.ld + rk.base, rk.step, t0, T, lt);
                xv.load(a.v + rv.base + me.slice * kSlice, rv.step, t0, T, lt);
                xd.load(a.dout + rv.base + me.slice * kSlice, rv.step, t0, T, lt);
                xs.load(a, me.tok0, me.h, t0, T, lt);
                xk.put_rows(buf + oK, t0, T, lt); xq.put_rows(buf + oQ, t0, T, lt);
                if constexpr (GLA) xa.put_rows_exp(buf + oA, t0, T, lt);
                xv.put(buf + oV, t0, T, lt); xd.put(buf + oDO, t0, T, lt);
                xs.put(buf + oSC, ha, t0, T, lt);
            }
            __syncthreads();
        }
        return;
    }
    float X[RT][CW];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const fc x = a.dsf ? *(const fc*)(a.dsf + ((size_t)me.bh * DK + me.rg * RT + r) * DV + me.col) : fc{0.f, 0.f};
#pragma unroll
        for (int j = 0; j < CW; ++j) X[r][j] = x[j];
    }
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
        const float* buf = lds + (c & 1) * kBuf;
#pragma unroll 4
        for (int i = kChunk - 1; i >= 0; --i) {
            const f4 sc = *(const f4*)(buf + oSC + kSc * i);
            const float gq = sc[0], gk = sc[1], ha = sc[2];
            float kf[RT], qf[RT], af[RT];
            get_rows<RT>(kf, buf + oK + i * DK + me.rg * 4);
            get_rows<RT>(qf, buf + oQ + i * DK + me.rg * 4);
            if constexpr (GLA) get_rows<RT>(af, buf + oA + i * DK + me.rg * 4);
            const int lc = i * kSlice + me.lcol;
            const fc vv = *(const fc*)(buf + oV + lc), dd = *(const fc*)(buf + oDO + lc);
            float du[CW] = {};
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int j = 0; j < CW; ++j) {
                    X[r][j] += qf[r] * (gq * dd[j]);
                    du[j] += kf[r] * X[r][j];
                    X[r][j] *= GLA ? af[r] : ha;
                }
            float pk = 0.f;
#pragma unroll
            for (int j = 0; j < CW; ++j) {
                du[j] = row_all(du[j]);
                pk += du[j] * vv[j];
            }
            pk = all_groups(pk);
            const int t = (nch - 1 - c) * kChunk + i;
            if (t < T) {
                if (me.lane == 0)
                    a.part_k[(size_t)(me.slice * kWaves + me.wave) * a.plane + (me.tok0 + t) * a.H + me.h] = pk;
                if (me.rg == 0) *(fc*)(a.dv + rv.base + (size_t)t * rv.step + me.col) = fc{gk * du[0], gk * du[1]};
            }
        }
        __syncthreads();
    }
    if (a.ds0) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
            *(fc*)(a.ds0 + ((size_t)me.bh * DK + me.rg * RT + r) * DV + me.col) = fc{X[r][0], X[r][1]};
    }
}

// ------------------------------------------------------------------------------------------------------------
// dq sweep (FWD: forward in time, S^T) and dk sweep (backward in time, X^T): rows are the dv value columns, a
// workgroup owns 64 key columns.  Tile element [r][j]: value column rg * RT + r, key column col + j.
//   FWD:   S^T = S^T diag(alpha) + (G^K v)^T k;   dq' = dout S^T;   dq = G^Q dq'
//   else:  X^T += (G^Q dout)^T q;   dk = G^K v X^T;   run += q dq - k dk;   X^T = X^T diag(alpha)
// ------------------------------------------------------------------------------------------------------------
template <bool GLA, int DK, int DV, bool FWD>
__device__ __forceinline__ void key_sweep(const FArgs& a, unsigned char* smem, int block, int grid) {
    constexpr int RT = DV / 16;
    constexpr bool NEED_DQ = GLA && !FWD;
    constexpr int oDO = 0, oV = oDO + kChunk * DV, oK = oV + kChunk * DV, oQ = oK + kChunk * kSlice,
                  oA = oQ + kChunk * kSlice, oDQ = oA + (GLA ? kChunk * kSlice : 0),
                  oSC = oDQ + (NEED_DQ ? kChunk * kSlice : 0), kBuf = oSC + kSc * kChunk;
    float* lds = (float*)smem;
    const Where me = where_segment(a, DK / kSlice, block, grid);
    if (me.bh < 0) return;
    const int T = me.T, nch = (T + kChunk - 1) / kChunk;
    const Rows rk = rows_of(a, me, DK), rv = rows_of(a, me, DV);
    if (me.wave >= kWaves) {
        const int lt = me.tid - 64 * kWaves;
        const float ha = head_alpha_of(a, me.h);
        const size_t ks = rk.base + me.slice * kSlice;
        for (int c = 0; c <= nch; ++c) {
            if (c < nch) {
                const int t0 = (FWD ? c : nch - 1 - c) * kChunk;
                float* buf = lds + (c & 1) * kBuf;
                RegsF<DV> xd, xv;
                RegsF<kSlice> xk, xq, xg;
                RegsA<kSlice> xa;
                RegsG xs;
                xd.load(a.dout + rv.base, rv.step, t0, T, lt); xv.load(a.v + rv.base, rv.step, t0, T, lt);
                xk.load(a.k + ks, rk.step, t0, T, lt); xq.load(a.q + ks, rk.step, t0, T, lt);
                if constexpr (GLA) xa.load(a.ld + ks, rk.step, t0, T, lt);
                if constexpr (NEED_DQ) xg.load(a.dq + ks, rk.step, t0, T, lt);
                xs.load(a, me.tok0, me.h, t0, T, lt);
                xd.put_rows(buf + oDO, t0, T, lt); xv.put_rows(buf + oV, t0, T, lt);
                xk.put(buf + oK, t0, T, lt); xq.put(buf + oQ, t0, T, lt);
                if constexpr (GLA) xa.put_exp(buf + oA, t0, T, lt);
                if constexpr (NEED_DQ) xg.put(buf + oDQ, t0, T, lt);
                xs.put(buf + oSC, ha, t0, T, lt);
            }
            __syncthreads();
        }
        return;
    }
    float M[RT][CW];
    const float* init = FWD ? a.s0 : a.dsf;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int j = 0; j < CW; ++j)
            M[r][j] = init ? init[((size_t)me.bh * DK + me.col + j) * DV + me.rg * RT + r] : 0.f;
    double run[CW] = {0.0, 0.0};  // dk sweep of GLA: rowsum(X_T' * S_T) + the sum of q dq - k dk over the tokens behind
    if constexpr (NEED_DQ) {
#pragma unroll
        for (int j = 0; j < CW; ++j) run[j] = (double)a.corr[(size_t)me.bh * DK + me.col + j];
    }
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
        const float* buf = lds + (c & 1) * kBuf;
#pragma unroll 4
        for (int ii = 0; ii < kChunk; ++ii) {
            const int i = FWD ? ii : kChunk - 1 - ii;
            const f4 sc = *(const f4*)(buf + oSC + kSc * i);
            const float gq = sc[0], gk = sc[1], ha = sc[2];
            float dd[RT], vv[RT];
            get_rows<RT>(dd, buf + oDO + i * DV + me.rg * 4);
            get_rows<RT>(vv, buf + oV + i * DV + me.rg * 4);
            const int lc = i * kSlice + me.lcol;
            const fc kf = *(const fc*)(buf + oK + lc), qf = *(const fc*)(buf + oQ + lc);
            fc al = fc{ha, ha};
            if constexpr (GLA) al = *(const fc*)(buf + oA + lc);
            const int t = (FWD ? c : nch - 1 - c) * kChunk + i;
            const size_t at = rk.base + (size_t)min(t, max(T - 1, 0)) * rk.step + me.col;
            float y[CW] = {};
            if constexpr (FWD) {
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int j = 0; j < CW; ++j) {
                        M[r][j] = __builtin_fmaf(M[r][j], al[j], (gk * vv[r]) * kf[j]);  // the state rounded once, not twice
                        y[j] += dd[r] * M[r][j];
                    }
                float pq = 0.f;
#pragma unroll
                for (int j = 0; j < CW; ++j) {
                    y[j] = row_all(y[j]);  // before the read gate: dG^Q = q . dq'
                    pq += qf[j] * y[j];
                }
                pq = all_groups(pq);
                if (t < T) {
                    if (me.lane == 0)
                        a.part_q[(size_t)(me.slice * kWaves + me.wave) * a.plane + (me.tok0 + t) * a.H + me.h] = pq;
                    if (me.rg == 0) *(fc*)(a.dq + at) = fc{gq * y[0], gq * y[1]};
                }
            } else {
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int j = 0; j < CW; ++j) {
                        M[r][j] += (gq * dd[r]) * qf[j];
                        y[j] += vv[r] * M[r][j];
                        M[r][j] *= al[j];
                    }
                fc dk;
#pragma unroll
                for (int j = 0; j < CW; ++j) dk[j] = gk * row_all(y[j]);
                if constexpr (NEED_DQ) {
                    const fc dqf = *(const fc*)(buf + oDQ + lc);
#pragma unroll
                    for (int j = 0; j < CW; ++j) run[j] += (double)qf[j] * (double)dqf[j] - (double)kf[j] * (double)dk[j];
                }
                if (t < T && me.rg == 0) {
                    *(fc*)(a.dk + at) = dk;
                    if constexpr (NEED_DQ) *(fc*)(a.dld + at) = fc{(float)run[0], (float)run[1]};
                }
            }
        }
        __syncthreads();
    }
    if constexpr (FWD && GLA) {  // rowsum(X_T' * S_T) for this lane's key columns
        float s[CW] = {};
        if (a.dsf) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int j = 0; j < CW; ++j)
                    s[j] += a.dsf[((size_t)me.bh * DK + me.col + j) * DV + me.rg * RT + r] * M[r][j];
        }
#pragma unroll
        for (int j = 0; j < CW; ++j) s[j] = row_all(s[j]);
        if (me.rg == 0) *(fc*)(a.corr + (size_t)me.bh * DK + me.col) = fc{s[0], s[1]};
    }
}

template <bool GLA, int DK, int DV>
__global__ __launch_bounds__(kThreads) void sla_bwd32_dv_kernel(const FArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    dv_sweep<GLA, DK, DV>(a, smem, (int)blockIdx.x, (int)gridDim.x);
}
template <bool GLA, int DK, int DV, bool FWD>
__global__ __launch_bounds__(kThreads) void sla_bwd32_key_kernel(const FArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    key_sweep<GLA, DK, DV, FWD>(a, smem, (int)blockIdx.x, (int)gridDim.x);
}
// The dq, the dv and, RetNet, the dk sweep side by side, DK / kSlice, DV / kSlice and DK / kSlice workgroups a sequence and
// head: none needs anything of the others (GLA's dk sweep makes the decay gradient from dq).  A sweep is bound by its serial
// walk over the tokens, so the chip has room for another one's workgroups: B=2 T=1021 H=8 64 x 128 GLA 122 -> 116 us for the
// backward pass, a training step of B=8 T=700 H=16 128 x 128 GLA 786 -> 707 us, of B=4 T=300 H=4 64 x 64 82 -> 73 us.
template <bool GLA, int DK, int DV>
constexpr int kSideBySide = (GLA ? 1 : 2) * (DK / kSlice) + DV / kSlice;
template <bool GLA, int DK, int DV>
__global__ __launch_bounds__(kThreads) void sla_bwd32_sweeps_kernel(const FArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int each = (int)gridDim.x / kSideBySide<GLA, DK, DV>, nk = each * (DK / kSlice), nv = each * (DV / kSlice);
    const int block = (int)blockIdx.x;
    if (block < nk)
        key_sweep<GLA, DK, DV, true>(a, smem, block, nk);
    else if (GLA || block < nk + nv)
        dv_sweep<GLA, DK, DV>(a, smem, block - nk, nv);
    else
        key_sweep<GLA, DK, DV, GLA>(a, smem, block - nk - nv, nk);
}

// ------------------------------------------------------------------------------------------------------------
// Pre-pass of the segment schedule (see launch_backward_f32): what a segment alone leaves behind.  blockIdx.y = 0,
// forward in time: the state at its end from a zero state; 1, backward in time: the cotangent of the state at its
// start when the one at its end is zero.  Both are M[key][value] with the decay per key, so both run on the tile of
// the key sweeps (rows: value columns, 64 key columns per workgroup); no sums across lanes.  `totals`: the segment's
// whole decay per key (the product the state itself would be multiplied by, factor by factor).
// ------------------------------------------------------------------------------------------------------------
template <bool GLA, int DK, int DV, bool FWD>
__device__ __forceinline__ void segment_alone(const FArgs& a, const Where& me, float* lds, float* end, float* totals) {
    constexpr int RT = DV / 16;
    constexpr int oR = 0, oC = oR + kChunk * DV, oA = oC + kChunk * kSlice, oSC = oA + (GLA ? kChunk * kSlice : 0),
                  kBuf = oSC + kSc * kChunk;
    const int T = me.T, nch = (T + kChunk - 1) / kChunk;
    const Rows rk = rows_of(a, me, DK), rv = rows_of(a, me, DV);
    if (me.wave >= kWaves) {
        const int lt = me.tid - 64 * kWaves;
        const float ha = head_alpha_of(a, me.h);
        const size_t ks = rk.base + me.slice * kSlice;
        for (int c = 0; c <= nch; ++c) {
            if (c < nch) {
                const int t0 = (FWD ? c : nch - 1 - c) * kChunk;
                float* buf = lds + (c & 1) * kBuf;
                RegsF<DV> xr;
                RegsF<kSlice> xc;
                RegsA<kSlice> xa;
                RegsG xs;
                xr.load((FWD ? a.v : a.dout) + rv.base, rv.step, t0, T, lt);
                xc.load((FWD ? a.k : a.q) + ks, rk.step, t0, T, lt);
                if constexpr (GLA) xa.load(a.ld + ks, rk.step, t0, T, lt);
                xs.load(a, me.tok0, me.h, t0, T, lt);
                xr.put_rows(buf + oR, t0, T, lt);
                xc.put(buf + oC, t0, T, lt);
                if constexpr (GLA) xa.put_exp(buf + oA, t0, T, lt);
                xs.put(buf + oSC, ha, t0, T, lt);
            }
            __syncthreads();
        }
        return;
    }
    float M[RT][CW] = {};
    fc total = {1.f, 1.f};
    __syncthreads();
    for (int c = 0; c < nch; ++c) {
        const float* buf = lds + (c & 1) * kBuf;
#pragma unroll 4
        for (int ii = 0; ii < kChunk; ++ii) {
            const int i = FWD ? ii : kChunk - 1 - ii;
            const f4 sc = *(const f4*)(buf + oSC + kSc * i);
            const float gate = FWD ? sc[1] : sc[0];
            float x[RT];
            get_rows<RT>(x, buf + oR + i * DV + me.rg * 4);
            const int lc = i * kSlice + me.lcol;
            const fc y = *(const fc*)(buf + oC + lc);
            fc al = fc{sc[2], sc[2]};
            if constexpr (GLA) al = *(const fc*)(buf + oA + lc);
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int j = 0; j < CW; ++j) {
                    if constexpr (FWD) {
                        M[r][j] = M[r][j] * al[j] + (gate * x[r]) * y[j];
                    } else {
                        M[r][j] += (gate * x[r]) * y[j];
                        M[r][j] *= al[j];
                    }
                }
            total *= al;  // a token past the end has factor 1
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < CW; ++j) {
        float* d = end + ((size_t)me.bh * DK + me.col + j) * DV + me.rg * RT;
#pragma unroll
        for (int r = 0; r < RT; r += 4) *(f4*)(d + r) = f4{M[r][j], M[r + 1][j], M[r + 2][j], M[r + 3][j]};
    }
    // the totals of segment 0 come from the forward half, the others from the backward half
    if (me.rg == 0 && FWD == (me.b % a.nseg == 0)) *(fc*)(totals + (size_t)me.bh * DK + me.col) = total;
}

template <bool GLA, int DK, int DV>
__global__ __launch_bounds__(kThreads) void sla_bwd32_segment_kernel(const FArgs a, float* states, float* cotangents,
                                                                      float* totals, bool want_ds0) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Where me = where_segment(a, DK / kSlice, (int)blockIdx.x, (int)gridDim.x);
    if (me.bh < 0) return;
    const int seg = me.b % a.nseg;
    if (blockIdx.y == 0) {
        if (seg == a.nseg - 1) return;  // nothing follows it
        segment_alone<GLA, DK, DV, true>(a, me, (float*)smem, states, totals);
    } else {
        if (seg == 0 && !want_ds0) return;  // nothing comes before it
        segment_alone<GLA, DK, DV, false>(a, me, (float*)smem, cotangents, totals);
    }
}

// Chains the segments: the recurrences are linear, so the state at a segment's end is its own plus its whole decay
// times the one it is entered with, and the same backward in time for the cotangents.  In place: `states` becomes the
// entry states, `cotangents` the cotangents at the segments' ends; ds0: the gradient of the initial state, or null.
// One thread per (batch row, head, key, four value columns) and direction (blockIdx.y).
__global__ __launch_bounds__(kEw) void sla_bwd32_chain_kernel(float* states, float* cotangents, const float* totals,
                                                              const float* s0, const float* dsf, float* ds0, int B, int H,
                                                              int dk, int dv, int nseg) {
    const size_t per_head = (size_t)dk * (dv / 4), idx = (size_t)blockIdx.x * kEw + threadIdx.x;
    if (idx >= (size_t)B * H * per_head) return;
    const size_t bh = idx / per_head, b = bh / H, h = bh % H, in = idx % per_head;
    const int d = (int)(in / (dv / 4));
    const size_t user = bh * dk * dv + in * 4;
    constexpr int kAtOnce = 8;  // only e and t are chained: what the segments left is loaded ahead of them
    auto seg_head = [&](int s) { return (b * nseg + s) * H + h; };
    auto at = [&](float* p, int s) { return p + seg_head(s) * dk * dv + in * 4; };
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    if (blockIdx.y == 0) {
        f4 e = s0 ? *(const f4*)(s0 + user) : zero;
        for (int s0 = 0; s0 < nseg; s0 += kAtOnce) {
            f4 x[kAtOnce];
            float D[kAtOnce];
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u) {  // the last segment's own slot and decay are not read (nseg >= 2)
                const int s = min(s0 + u, nseg - 2);
                x[u] = *(const f4*)at(states, s);
                D[u] = totals[seg_head(s) * dk + d];
            }
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u) {
                if (s0 + u >= nseg) break;
                *(f4*)at(states, s0 + u) = e;
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = x[u][i] + D[u] * e[i];
            }
        }
    } else {
        f4 t = dsf ? *(const f4*)(dsf + user) : zero;
        const int lowest = ds0 ? 0 : 1;  // the first segment's start cotangent exists only if it is wanted
        for (int s0 = nseg - 1; s0 >= 0; s0 -= kAtOnce) {
            f4 x[kAtOnce];
            float D[kAtOnce];
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u) {
                const int s = max(s0 - u, lowest);
                x[u] = *(const f4*)at(cotangents, s);
                D[u] = totals[seg_head(s) * dk + d];
            }
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u) {
                if (s0 - u < 0) break;
                *(f4*)at(cotangents, s0 - u) = t;
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = x[u][i] + D[u] * t[i];
            }
        }
        if (ds0) *(f4*)(ds0 + user) = t;
    }
}

template <typename K>
bool allow_lds(K kernel, int lds) {
    if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess)
        return true;
    (void)hipGetLastError();
    return false;
}

struct Segments {  // buffers of the segment schedule, see launch_backward_f32
    float* states;
    float* cotangents;
    float* totals;
};

template <bool GLA, int DK, int DV>
int launch_sweeps(FArgs a, const Segments& sg, bool state_only, hipStream_t stream) {
    constexpr int ldsS = 2 * 4 * (kChunk * DV + (GLA ? 2 : 1) * kChunk * kSlice + kSc * kChunk);
    constexpr int ldsV = 2 * 4 * ((GLA ? 3 : 2) * kChunk * DK + 2 * kChunk * kSlice + kSc * kChunk);
    constexpr int ldsQ = 2 * 4 * (2 * kChunk * DV + (GLA ? 3 : 2) * kChunk * kSlice + kSc * kChunk);
    constexpr int ldsK = 2 * 4 * (2 * kChunk * DV + (GLA ? 4 : 2) * kChunk * kSlice + kSc * kChunk);
    // One launch for several sweeps where its workgroups' larger LDS still lets two share a compute unit (ldsK is ldsQ for
    // RetNet, whose dk sweep is among them).
    constexpr int ldsVQ = ldsV > ldsQ ? ldsV : ldsQ;
    constexpr bool kTogether = ldsVQ <= 80 * 1024;
    static_assert(ldsV <= 160 * 1024 && ldsQ <= 160 * 1024 && ldsK <= 160 * 1024, "fits the LDS of a compute unit");
    // once per device and instantiation (bit d = done on device d); not a stream operation
    static std::atomic<uint64_t> configured{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return SLA_ERR_HIP;
    }
    if (!((configured.load(std::memory_order_acquire) >> dev) & 1u)) {
        if (!allow_lds(sla_bwd32_dv_kernel<GLA, DK, DV>, ldsV) ||
            !allow_lds(sla_bwd32_key_kernel<GLA, DK, DV, true>, ldsQ) ||
            !allow_lds(sla_bwd32_key_kernel<GLA, DK, DV, false>, ldsK) ||
            !allow_lds(sla_bwd32_segment_kernel<GLA, DK, DV>, ldsS) || !allow_lds(sla_bwd32_sweeps_kernel<GLA, DK, DV>, ldsVQ))
            return SLA_ERR_HIP;
        configured.fetch_or(uint64_t(1) << dev, std::memory_order_release);
    }
    const unsigned bh = (unsigned)(a.B * a.H);
    const dim3 block(kThreads);
    auto grid = [bh](unsigned slices) { return dim3(((bh + 7u) / 8u) * 8u * slices); };  // see tok::where()
    if (a.nseg > 1) {
        dim3 g = grid(DK / kSlice);
        g.y = 2;
        hipLaunchKernelGGL((sla_bwd32_segment_kernel<GLA, DK, DV>), g, block, (size_t)ldsS, stream, a, sg.states,
                           sg.cotangents, sg.totals, a.ds0 != nullptr);
        const int rows = a.B / a.nseg;
        const size_t n = (size_t)rows * a.H * DK * (DV / 4);
        hipLaunchKernelGGL(sla_bwd32_chain_kernel, dim3((unsigned)((n + kEw - 1) / kEw), 2), dim3(kEw), 0, stream,
                           sg.states, sg.cotangents, (const float*)sg.totals, a.s0, a.dsf, a.ds0, rows, a.H, DK, DV,
                           a.nseg);
        if (hipGetLastError() != hipSuccess) return SLA_ERR_HIP;
        a.s0 = sg.states;
        a.dsf = sg.cotangents;
        a.ds0 = nullptr;
    }
    if (kTogether && !state_only) {
        hipLaunchKernelGGL((sla_bwd32_sweeps_kernel<GLA, DK, DV>), grid(kSideBySide<GLA, DK, DV>), block, (size_t)ldsVQ, stream,
                           a);
    } else {
        hipLaunchKernelGGL((sla_bwd32_dv_kernel<GLA, DK, DV>), grid(DV / kSlice), block, (size_t)ldsV, stream, a);
        if (!state_only)
            hipLaunchKernelGGL((sla_bwd32_key_kernel<GLA, DK, DV, true>), grid(DK / kSlice), block, (size_t)ldsQ, stream, a);
    }
    if (!state_only && (GLA || !kTogether)) {
        hipLaunchKernelGGL((sla_bwd32_key_kernel<GLA, DK, DV, false>), grid(DK / kSlice), block, (size_t)ldsK, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SLA_OK : SLA_ERR_HIP;
}

template <bool GLA, int DK>
int launch_dv(const FArgs& a, const Segments& sg, int dv, bool state_only, hipStream_t stream) {
    switch (dv) {
        case 64: return launch_sweeps<GLA, DK, 64>(a, sg, state_only, stream);
        case 128: return launch_sweeps<GLA, DK, 128>(a, sg, state_only, stream);
        case 256: return launch_sweeps<GLA, DK, 256>(a, sg, state_only, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}

template <bool GLA>
int launch_dk(const FArgs& a, const Segments& sg, int dk, int dv, bool state_only, hipStream_t stream) {
    switch (dk) {
        case 64: return launch_dv<GLA, 64>(a, sg, dv, state_only, stream);
        case 128: return launch_dv<GLA, 128>(a, sg, dv, state_only, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}

// Segments per batch row.  A sweep is a serial walk of about 0.3 us a token in every workgroup, so few sequences leave
// most of the chip idle: rows are cut until the narrowest sweep has a workgroup for each of 256 compute units, into
// segments of at least 32 tokens.  Heads up to 64 x 128 take half the vector work per token, so two workgroups share a
// compute unit to gain and 512 are wanted, but not with segments under 64 tokens, where the pre-pass and the chain cost
// more than that gives.  Call in us (a launch for every sweep), one pass -> 256 wanted / 512 wanted:
//     B=2 T=1021 H=8  64 x 128    917 -> 141 / 150           B=6 T=1500 H=16 64 x 64    1000 -> 602 / 397
//     B=1 T=300  H=4  64 x 64     215 -> 52 (64 tokens: 76)  B=7 T=1000 H=16 64 x 128    921 -> 697 / 641
//     B=1 T=4096 H=2  128 x 128  3827 -> 139 / 149           B=4 T=2048 H=5  128 x 256  2548 -> 758 / 802
//     B=5 T=300  H=12 128 x 256   421 -> 368 / 410           B=8 T=700  H=16 128 x 128   708 (one pass) / 790
// Rows of up to 128 tokens stay in one pass and in the workspace it takes: such a call is 0.15 ms at most.
// Packed batches run in one pass (their lengths are known on the device only), and so does p.segments == 1: the caller's
// workspace has no room for more.
int segments_of(const sla_params& p, bool packed, int* seg_len) {
    constexpr int kShortest = 32, kOnePass = 128;
    *seg_len = p.T;
    const size_t groups = (size_t)p.B * p.H * ((p.dk < p.dv ? p.dk : p.dv) / kSlice);
    if (packed || p.segments == 1 || groups == 0 || p.T <= kOnePass) return 1;
    const size_t target = p.dk * p.dv <= 64 * 128 && groups * p.T >= 512 * 64 ? 512 : 256;
    if (2 * groups > target) return 1;
    const int want = (int)(target / groups);
    int len = ((p.T + want - 1) / want + kChunk - 1) / kChunk * kChunk;
    if (len < kShortest) len = kShortest;
    *seg_len = len;
    return (p.T + len - 1) / len;
}

size_t round4(size_t n) { return (n + 3) & ~(size_t)3; }

}  // namespace

// Workspace, in floats: gates 2 [B,T,H]; dk/8 partial planes of dG^Q and dv/8 of dG^K (one per compute wave and
// slice); for GLA rowsum(X_T' * S_T) [B,H,dk] (per segment); with nseg > 1 segments per batch row also their states and
// cotangents 2 [B,nseg,H,dk,dv] and their decays [B,nseg,H,dk].
size_t backward_f32_workspace_floats(const sla_params& p, bool packed) {
    const size_t rows = packed ? (size_t)p.T : (size_t)p.B * p.T, n = round4(rows * p.H);
    int len = 0;
    const size_t nseg = segments_of(p, packed, &len), heads = (size_t)p.B * nseg * p.H;
    return n * (2 + (size_t)p.dk / (4 * CW) + (size_t)p.dv / (4 * CW)) +
           (p.variant == SLA_GLA ? round4(heads * p.dk) : 0) +
           (nseg > 1 ? 2 * heads * p.dk * p.dv + round4(heads * p.dk) : 0);
}

// One pass, or -- few sequences, see segments_of() -- every batch row in nseg segments that run side by side:
//   1. what each segment alone leaves behind, forward (its state) and backward (its cotangent), in one launch;
//   2. the chain kernel turns those into every segment's entry state and end cotangent;
//   3. the three sweeps over B * nseg sequences.  The decay gradient's running sum starts, per segment, from
//      rowsum(cotangent * state) at its end, the same identity as at the end of a whole sequence.
// All of it in fp32 and with the decay applied token by token, so the domain is that of the single pass.
int launch_backward_f32(const sla_params& p, const void* q, const void* k, const void* v, const float* ql,
                        const float* kl, const void* ld, const float* s0, const void* dout, const float* dsf, void* dq,
                        void* dk, void* dv, float* dql, float* dkl, void* dld, float* ds0, float* ws, const int* cu,
                        hipStream_t stream) {
    const size_t rows = cu ? (size_t)p.T : (size_t)p.B * p.T, n = round4(rows * p.H);
    const int pq = p.dk / (4 * CW), pv = p.dv / (4 * CW);
    FArgs a;
    a.q = (const float*)q; a.k = (const float*)k; a.v = (const float*)v; a.dout = (const float*)dout;
    a.ld = p.variant == SLA_GLA ? (const float*)ld : nullptr;
    a.ld_head = p.variant == SLA_RETNET ? (const float*)ld : nullptr;
    a.s0 = s0; a.dsf = dsf;
    a.dq = (float*)dq; a.dk = (float*)dk; a.dv = (float*)dv; a.dld = (float*)dld; a.ds0 = ds0;
    float* w = ws;
    float* gq = w; w += n;
    float* gk = w; w += n;
    a.gq = gq; a.gk = gk;
    a.part_q = w; w += n * pq;
    a.part_k = w; w += n * pv;
    int seg_len = 0;
    const int nseg = segments_of(p, cu != nullptr, &seg_len);
    const size_t heads = (size_t)p.B * nseg * p.H;
    a.corr = w;
    if (p.variant == SLA_GLA) w += round4(heads * p.dk);
    Segments sg = {nullptr, nullptr, nullptr};
    if (nseg > 1) {
        sg.states = w; w += heads * p.dk * p.dv;
        sg.cotangents = w; w += heads * p.dk * p.dv;
        sg.totals = w;
    }
    a.nseg = nseg; a.seg_len = seg_len;
    a.plane = n; a.rows = rows; a.cu = cu;
    a.B = p.B * nseg; a.T = p.T; a.H = p.H;
    a.head_major = (p.flags & SLA_FLAG_HEAD_MAJOR) != 0;
    const bool state_only = rows == 0;  // no tokens: the final state's cotangent is the initial state's
    int rc = launch_bwd_gates(ql, kl, gq, gk, rows, p.H, stream);
    if (rc != SLA_OK) return rc;
    rc = p.variant == SLA_GLA ? launch_dk<true>(a, sg, p.dk, p.dv, state_only, stream)
                              : launch_dk<false>(a, sg, p.dk, p.dv, state_only, stream);
    if (rc != SLA_OK || state_only) return rc;
    return launch_bwd_logits(GateGrad{gq, a.part_q, pq, n, dql}, GateGrad{gk, a.part_k, pv, n, kl ? dkl : nullptr}, rows,
                             p.H, cu, p.B, stream);
}

}  // namespace sla
