// Backward pass of the gated delta rule on bf16 tensors, chunk-parallel.  Only res_t (forward in time) and du_t (backward)
// depend on a state through the rule's own feedback; the sweeps of sla_backward_gdn_block.hip find them, both in one launch,
// and keep for every 64-token chunk the state S entering it and the cotangent X of the state behind it.  With res and du
// known every recurrence is linear and all gradients of a chunk depend on its own rows, S and X: one workgroup per chunk and
// head makes them.  With c_t the running log-decay of the chunk, p = e^c, A its total, D[t][j] = p_t / p_j (j <= t),
// u = beta res, w = beta du:
//     N'[t][j] = D (dout_t . u_j), j <= t      M[t][j] = -D (w_t . u_j), j < t
//     dq'_t = p_t dout_t S^T + sum_j N'[t][j] k_j                                   dq = G^Q dq'    dG^Q = q . dq'
//     dk_t  = (A / p_t) u_t X^T - p_t w_t S^T + sum_j (M + M^T)[t][j] k_j + sum_s N'[s][t] G^Q_s q_s
//     dv = G^K w    dG^K = w . v    dbeta = du . res
//     dlog_decay_t = <X, S_end> + sum_{s >= t} (G^Q dG^Q - G^K dG^K)_s
// (the block form's lines, see sla_backward_gdn_block.hip, which hold for any length of block once u and w are known).
// Every factor is <= 1.  The suffix sums of the decay gradient run afterwards over spans of 512 tokens, each from <X, S_end>
// at their ends (kGdnAnchor in sla_gdn_block.h), which has nothing to average a rounding over: both states are
// taken there as two bf16 parts, 2^-17 off fp32, and at the sequence's end in fp32 by the state sweep.  (From the bf16 states
// alone the last token's gradient was 2.0e-3 off at T = 8 with states in and out, 2.3e-4 from the sweeps.)
// Against the four sweeps of sla_backward_gdn_block.hip, a backward call: few sequences 1.6 to 3.8 times (B=2 T=4096 H=4 128 x 256
// 1020 -> 266 us, B=2 T=1000 H=8 128 x 128 227 -> 94, B=1 T=300 H=4 104 -> 53, 4096 packed tokens H=8 141 -> 86), where the sweeps
// leave some compute units idle 1.1 to 1.25 times (B=8 T=4096 H=12 866 -> 783, 64 x 128 heads H=16 832 -> 674); where they fill the
// chip see gdn_sweeps_are_faster().  Two sweeps 424 us and this kernel 439 at B=8 T=4096 H=16 128 x 128.  No output is
// further from fp32 tensors than theirs (dk 4.1e-3 -> 3.4e-3, dv 3.4e-3 -> 3.0e-3, dlog_decay
// 3.0e-2 -> 2.2e-2, dbeta the same): du stays in fp32, so that dbeta and w are what they were.
#include <hip/hip_runtime.h>
#include <stdint.h>


#include "sla.h"
#include "sla_chunk.h"
#include "sla_chunk_plan.h"
#include "sla_gate_grad.h"
#include "sla_gdn_block.h"

namespace sla {

int launch_bwd_gates(const float* ql, const float* kl, float* gq, float* gk, size_t rows, int H, hipStream_t stream);

namespace chk {

static_assert(kChunk == kGdnChunk, "the sweeps keep a state per chunk");

constexpr int kThreads = 256;
constexpr int kSpanChunks = kGdnAnchor / kChunk;

struct GdnArgs {
    Args a;  // gq, gk: the gates; dgq, dgk: their gradients; S, X and the decays are below
    const uint16_t* S;    // [slot][H][dv][dk], see keep_state()
    const uint16_t* X;
    const uint16_t* Srest;  // [rows / 512 + 1][H][dv][dk] what rounding left of S and X at every 512th token of a sequence
    const uint16_t* Xrest;
    const uint16_t* res;  // [rows,H,dv]
    const float* du;
    const float* ld;      // [rows,H]
    const float* beta;
    float* e;             // [rows,H] the scalars whose suffix sums dlog_decay is
    float* anchor;        // [rows / 512 + 1][H][8] <X, S> at every 512th token of a sequence, an eighth of the value columns each
    float* dbeta;
};

// Four waves.  For dq and dk a wave takes 32 key dimensions and TB = DK / 32 of the four token blocks.  LDS in bytes: two
// workgroups share a compute unit.
template <int DK>
struct GLds {
    static constexpr int WD = DK / 32, WT = 4 / WD, TB = WD;
    static constexpr int rows = kChunk * DK * 2;
    static constexpr int SS = DK + 16;                  // row stride of S and X, elements: read by columns
    static constexpr int state = 32 * SS * 2, slab = kChunk * 64, matrix = kChunk * kChunk * 2;
    static constexpr int oQ = 0, oK = oQ + rows;
    static constexpr int oS = oK + rows, oX = oS + state;                     // 32 value columns at a time: S, X,
    static constexpr int oO = oX + state, oR = oO + slab, oD = oR + slab;     // dout, res, w
    static constexpr int oN = oS, oN2 = oN + matrix, oM = oN2 + matrix;       // after them: N', its transpose by G^Q, M + M^T
    static constexpr int oSc = std::max(oD + slab, oM + matrix);              // per token: G^Q, G^K, beta, c, du.res, w.v
    static constexpr int oRed = oSc + 6 * kChunk * 4;                         // partial dG^Q [WD][64], <X, S_end> [4]
    static constexpr int total = oRed + WD * kChunk * 4 + 16;
    static_assert(total <= 80 * 1024, "two workgroups per compute unit");
};

template <int DK, int DV>
__global__ __launch_bounds__(kThreads, 2) void sla_chunk_gdn_kernel(const GdnArgs ga) {
    typedef GLds<DK> L;
    constexpr int WD = L::WD, TB = L::TB, U = DK / 8, NS = DV / 32, NM = 3, NU = DK / 64;
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t* sq = (uint16_t*)(smem + L::oQ);
    uint16_t* sk = (uint16_t*)(smem + L::oK);
    uint16_t* sS = (uint16_t*)(smem + L::oS);
    uint16_t* sX = (uint16_t*)(smem + L::oX);
    uint16_t* so = (uint16_t*)(smem + L::oO);
    uint16_t* sr = (uint16_t*)(smem + L::oR);
    uint16_t* sd = (uint16_t*)(smem + L::oD);
    uint16_t* sn = (uint16_t*)(smem + L::oN);
    uint16_t* sn2 = (uint16_t*)(smem + L::oN2);
    uint16_t* sm = (uint16_t*)(smem + L::oM);
    float* sgq = (float*)(smem + L::oSc);
    float* sgk = sgq + kChunk;
    float* sbeta = sgk + kChunk;
    float* sc = sbeta + kChunk;
    float* spb = sc + kChunk;
    float* spk = spb + kChunk;
    float* sred = (float*)(smem + L::oRed);
    float* sphi = sred + WD * kChunk;
    const Args& a = ga.a;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wd = w % WD, wt = w / WD;

    // Chunk and head, as in sla_chunk_backward_kernel.
    const int per = (int)(gridDim.x >> 3), id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (id >= a.slots * a.H) return;
    const int h = id % a.H, slot = id / a.H;
    int b, chunk;
    if (!chunk_of(a, slot, b, chunk)) return;
    const Sequence s = sequence(a, b);
    const int t0 = chunk * kChunk, len = min(kChunk, s.T - t0);
    const Rows rq = rows_of<DK>(a, a.q, s, b, h), rk = rows_of<DK>(a, a.k, s, b, h);
    const Rows rv = rows_of<DV>(a, a.v, s, b, h), ro = rows_of<DV>(a, a.dout, s, b, h);
    const Rows rr = rows_of<DV>(a, ga.res, s, b, h);
    // (under 2^31 bytes: a sequence's states of both kinds are dk / 64 times as many and more, a GiB at most)
    const Rows rd = {__builtin_amdgcn_make_buffer_rsrc((void*)(ga.du + s.tok0 * a.H * DV), 0, s.T * a.H * DV * 4, kRsrcWord3),
                     h * DV * 4, a.H * DV * 4};
    const Rows rdv = rows_of<DV>(a, a.dv, s, b, h);
    const size_t state = ((size_t)slot * a.H + h) * (size_t)(DK * DV);
    const int d0 = 32 * wd + 8 * g, m0 = TB * wt;  // this lane's eight key dimensions; its tokens 16 m + r, m0 <= m < m0 + TB

    // Rows of 32 value columns: thread (token tid / 4, 8 columns), bf16 two steps at once (whole 128-byte lines); 32 rows of S, X.
    struct Pre {
        u4 o[2], rs[2], v[2], du[2], S[NU], X[NU];  // du: 8 columns of one step
    } pre;
    const int tok = tid >> 2, unit = tid & 3;
    auto load_rows = [&](int c) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int col = 32 * (c + i) + 8 * unit;
            pre.o[i] = ro.load(t0 + tok, col);
            pre.rs[i] = rr.load(t0 + tok, col);
            pre.v[i] = rv.load(t0 + tok, col);
        }
    };
    auto load_states = [&](int c) {
#pragma unroll
        for (int i = 0; i < 2; ++i) pre.du[i] = rd.load(t0 + tok, 2 * (32 * c + 8 * unit + 4 * i));  // in 2-byte columns
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const size_t at = state + (size_t)c * (32 * DK) + 8 * (tid + kThreads * i);
            pre.S[i] = __builtin_nontemporal_load((const u4*)(ga.S + at));
            pre.X[i] = __builtin_nontemporal_load((const u4*)(ga.X + at));
        }
    };
    {
        u4 qx[TB], kx[TB];
#pragma unroll
        for (int m = 0; m < TB; ++m) {
            qx[m] = rq.load(t0 + 16 * (m0 + m) + r, d0);
            kx[m] = rk.load(t0 + 16 * (m0 + m) + r, d0);
        }
        load_rows(0);
        load_states(0);
        if (w == 0) {
            sgq[lane] = load_scalar(scalars_of(a, a.gq, s, h), t0 + lane);
            sgk[lane] = load_scalar(scalars_of(a, a.gk, s, h), t0 + lane);
            sbeta[lane] = load_scalar(scalars_of(a, ga.beta, s, h), t0 + lane);
            float c = load_scalar(scalars_of(a, ga.ld, s, h), t0 + lane) * kLog2e;
#pragma unroll
            for (int d = 1; d < kChunk; d *= 2) {
                const float x = __shfl_up(c, d);
                if (lane >= d) c += x;
            }
            sc[lane] = c;
        }
#pragma unroll
        for (int m = 0; m < TB; ++m) {
            const int at = 8 * unit_at<U>(16 * (m0 + m) + r, 4 * wd + g);
            *(u4*)(sq + at) = qx[m];
            *(u4*)(sk + at) = kx[m];
        }
    }

    // ---- the value columns, 32 at a time: dout S^T, res X^T, w S^T, dout . res, w . res, and dv
    f4 aq[TB][2], ak[TB][2], aw[TB][2], N[NM], M[NM];
#pragma unroll
    for (int m = 0; m < TB; ++m)
#pragma unroll
        for (int i = 0; i < 2; ++i) aq[m][i] = ak[m][i] = aw[m][i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < NM; ++x) N[x] = M[x] = f4{0.f, 0.f, 0.f, 0.f};
    float pb = 0.f, pk = 0.f;                                       // this thread's share of du . res, w . v of its token
    for (int c2 = 0; c2 < NS; c2 += 2)
#pragma unroll
    for (int x2 = 0; x2 < 2; ++x2) {
        const int c = c2 + x2;
        __syncthreads();  // the readers of what lies here are done; the scalars are in LDS
        const int at = 8 * unit_at<4>(tok, unit);
        *(u4*)(so + at) = pre.o[x2];
        *(u4*)(sr + at) = pre.rs[x2];
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int j = tid + kThreads * i, place = (j / U) * L::SS + 8 * (j % U);
            *(u4*)(sS + place) = pre.S[i];
            *(u4*)(sX + place) = pre.X[i];
        }
        {
            const float gk = sgk[tok], beta = sbeta[tok];
            f4 x[2];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = __uint_as_float(pre.du[e >> 2][e & 3]);
                pb = fmaf(d, bf_at(pre.rs[x2], e), pb);
                x[e >> 2][e & 3] = beta * d;
                pk = fmaf(x[e >> 2][e & 3], bf_at(pre.v[x2], e), pk);
            }
            *(u4*)(sd + at) = pack8(x[0], x[1]);
            rdv.put(t0 + tok, 32 * c + 8 * unit, pack8(x[0] * gk, x[1] * gk));
        }
        if (x2 == 1 && c + 1 < NS) load_rows(c + 1);
        if (c + 1 < NS) load_states(c + 1);
        __syncthreads();
        s8 fS[2], fX[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int G = 2 * (r & 3) + i, from = (8 * g + (r >> 2)) * L::SS + 32 * wd + 4 * (2 * (G & 3) + (G >> 2));
            fS[i] = join(lds_tr(sS + from), lds_tr(sS + from + 4 * L::SS));
            fX[i] = join(lds_tr(sX + from), lds_tr(sX + from + 4 * L::SS));
        }
        auto slab = [&](const uint16_t* x, int row) { return op(*(const u4*)(x + 8 * unit_at<4>(row, g))); };
#pragma unroll
        for (int m = 0; m < TB; ++m) {
            const int row = 16 * (m0 + m) + r;
            const s8 fo = slab(so, row), fr = slab(sr, row), fd = slab(sd, row);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                mma(aq[m][i], fS[i], fo);
                mma(ak[m][i], fX[i], fr);
                mma(aw[m][i], fS[i], fd);
            }
        }
#pragma unroll
        for (int x = 0; x < NM; ++x) {
            const int tile = w + 4 * x;
            if (tile < 10) {
                const int t = 16 * (int)((kTileT >> (4 * tile)) & 15) + r;
                const s8 fr = slab(sr, 16 * (int)((kTileJ >> (4 * tile)) & 15) + r);
                mma(N[x], slab(so, t), fr);
                mma(M[x], slab(sd, t), fr);
            }
        }
    }
    pb += dpp<0xB1>(pb);  // the four threads of a token
    pb += dpp<0x4E>(pb);
    pk += dpp<0xB1>(pk);
    pk += dpp<0x4E>(pk);
    if (unit == 0) {
        spb[tok] = pb;
        spk[tok] = pk;
    }
    __syncthreads();

    // ---- N', G^Q N'^T, M + M^T
    auto n_at = [&](uint16_t* x, int row, int col) { return x + 8 * unit_at<8>(row, col >> 3) + (col & 7); };
    const float c_end = sc[kChunk - 1];
#pragma unroll
    for (int x = 0; x < NM; ++x) {
        const int tile = w + 4 * x;
        if (tile < 10) {
            const int tb = 16 * (int)((kTileT >> (4 * tile)) & 15), j = 16 * (int)((kTileJ >> (4 * tile)) & 15) + r;
            const f4 gq = *(const f4*)(sgq + tb + 4 * g), ct = *(const f4*)(sc + tb + 4 * g);
            const float cj = sc[j], bj = sbeta[j];
            f4 n2, m2;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = tb + 4 * g + e;
                const float D = ex2(fminf(ct[e] - cj, 0.f)) * bj;
                const float y = t >= j ? N[x][e] * D : 0.f;  // the first four tiles are the diagonal's
                n2[e] = y * gq[e];
                m2[e] = t > j ? -M[x][e] * D : 0.f;
                *n_at(sn, t, j) = (uint16_t)pack2(y, 0.f);
                if (x > 0 || t >= j) *n_at(sm, t, j) = (uint16_t)pack2(m2[e], 0.f);
                if (x == 0 && t > j) *n_at(sm, j, t) = (uint16_t)pack2(m2[e], 0.f);
            }
            *(u2*)n_at(sn2, j, tb + 4 * g) = pack4(n2);
            if (x > 0) *(u2*)n_at(sm, j, tb + 4 * g) = pack4(m2);
        }
    }
    for (int x = tid; x < 128; x += kThreads) {  // the products take 32 tokens at a time: the tiles above the diagonal inside them
        const int blk = x >> 6, row = (x & 63) >> 2, col = 4 * (x & 3);
        *(u2*)n_at(sn, 32 * blk + row, 32 * blk + 16 + col) = u2{0u, 0u};
        *(u2*)n_at(sn2, 32 * blk + 16 + row, 32 * blk + col) = u2{0u, 0u};
    }
    __syncthreads();

    // ---- dq, dk of the wave's 32 dimensions.  Columns of a [token][DK] array: slots 8g .. 8g + 7 are rows `row0` ..
    auto col_op = [&](const uint16_t* x, int row0, int i) {
        const int row = row0 + (r >> 2);
        return join(lds_tr(x + 8 * unit_at<U>(row, 4 * wd + (r & 3)) + 4 * i), lds_tr(x + 8 * unit_at<U>(row + 4, 4 * wd + (r & 3)) + 4 * i));
    };
    auto n_op = [&](uint16_t* x, int row, int col) { return op(*(const u4*)n_at(x, row, col)); };
    auto put_row = [&](uint16_t* x, int t, f4 lo, f4 hi) { rows_of<DK>(a, x, s, b, h).put(t0 + t, d0, pack8(lo, hi)); };
    s8 fk[2][2], fq[2][2];  // 32 tokens pp, tile i
#pragma unroll
    for (int pp = 0; pp < 2; ++pp)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            fk[pp][i] = col_op(sk, 32 * pp + 8 * g, i);
            fq[pp][i] = col_op(sq, 32 * pp + 8 * g, i);
        }
#pragma unroll
    for (int mm = 0; mm < TB; ++mm) {
        const int m = m0 + mm, t = 16 * m + r;
        const u4 qx = *(const u4*)(sq + 8 * unit_at<U>(t, 4 * wd + g));
        const float gq = sgq[t], ct = sc[t], p = ex2(ct), fx = sbeta[t] * ex2(fminf(c_end - ct, 0.f));
        f4 q2[2], k2[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            q2[i] = aq[mm][i] * p;
            k2[i] = ak[mm][i] * fx - aw[mm][i] * p;
        }
#pragma unroll
        for (int pp = 0; pp < 2; ++pp) {
            const s8 mo = n_op(sm, t, 32 * pp + 8 * g);
#pragma unroll
            for (int i = 0; i < 2; ++i) mma(k2[i], fk[pp][i], mo);
            if (32 * pp + 16 >= 16 * m) {
                const s8 n = n_op(sn2, t, 32 * pp + 8 * g);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(k2[i], fq[pp][i], n);
            }
            if (32 * pp <= 16 * m) {
                const s8 n = n_op(sn, t, 32 * pp + 8 * g);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(q2[i], fk[pp][i], n);
            }
        }
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sum = fmaf(bf_at(qx, e), q2[e >> 2][e & 3], sum);
        sum = all_groups(sum);
        if (g == 0) sred[wd * kChunk + t] = sum;
        put_row(a.dk, t, k2[0], k2[1]);
        put_row(a.dq, t, q2[0] * gq, q2[1] * gq);
    }
    // <X, S> at the end of the 512-token span: the span's eight chunks make an eighth each (in the last one alone it was a
    // tail of 8 us, 128 x 256).  The states of both sides are in the same order.
    const int last = chunk | (kSpanChunks - 1), part = chunk & (kSpanChunks - 1);
    const bool anchored = (last + 1) * kChunk < s.T;
    const size_t aid = (s.tok0 + (size_t)(last + 1) * kChunk) / kGdnAnchor;
    if (anchored) {
        constexpr int kUnits = DK * DV / 8 / kSpanChunks;
        const u4* X = (const u4*)(ga.X + state + (size_t)(last - chunk) * a.H * (DK * DV)) + part * kUnits;
        const u4* S = (const u4*)(ga.S + state + (size_t)(last - chunk + 1) * a.H * (DK * DV)) + part * kUnits;
        const u4* Xr = (const u4*)(ga.Xrest + (aid * a.H + h) * (size_t)(DK * DV)) + part * kUnits;
        const u4* Sr = (const u4*)(ga.Srest + (aid * a.H + h) * (size_t)(DK * DV)) + part * kUnits;
        float phi = 0.f;
#pragma unroll
        for (int i = tid; i < kUnits; i += kThreads) {
            const u4 s0 = S[i], s1 = Sr[i], x0 = X[i], x1 = Xr[i];
#pragma unroll
            for (int e = 0; e < 8; ++e) phi = fmaf(bf_at(s0, e) + bf_at(s1, e), bf_at(x0, e) + bf_at(x1, e), phi);
        }
        phi = all_groups(row_all(phi));
        if (lane == 0) sphi[w] = phi;
    }
    __syncthreads();
    if (w == 0) {
        float dgq = 0.f;
#pragma unroll
        for (int n = 0; n < WD; ++n) dgq += sred[n * kChunk + lane];
        const float dgk = spk[lane];
        if (lane < len) {
            const size_t at = (s.tok0 + t0 + lane) * a.H + h;
            a.dgq[at] = dgq;
            a.dgk[at] = dgk;
            ga.dbeta[at] = spb[lane];
            ga.e[at] = sgq[lane] * dgq - sgk[lane] * dgk;
        }
        if (lane == 0 && anchored)
            ga.anchor[(aid * a.H + h) * kSpanChunks + part] = (sphi[0] + sphi[1]) + (sphi[2] + sphi[3]);
    }
}

template <int DK, int DV>
static int launch_gdn_chunks(const GdnArgs& ga, hipStream_t stream) {
    if (!allow_lds<sla_chunk_gdn_kernel<DK, DV>>(GLds<DK>::total)) return SLA_ERR_HIP;
    const unsigned n = ((unsigned)ga.a.slots * ga.a.H + 7u) / 8u * 8u;
    hipLaunchKernelGGL((sla_chunk_gdn_kernel<DK, DV>), dim3(n), dim3(kThreads), (size_t)GLds<DK>::total, stream, ga);
    return hipGetLastError() == hipSuccess ? SLA_OK : SLA_ERR_HIP;
}
template <int DK>
static int launch_gdn_chunks_dv(const GdnArgs& ga, int dv, hipStream_t stream) {
    switch (dv) {
        case 64: return launch_gdn_chunks<DK, 64>(ga, stream);
        case 128: return launch_gdn_chunks<DK, 128>(ga, stream);
        case 256: return launch_gdn_chunks<DK, 256>(ga, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}

}  // namespace chk

int launch_backward_gdn_chunks(const sla_params& p, const void* q, const void* k, const void* v, const float* ql,
                               const float* kl, const float* ld, const float* beta, const float* s0, const void* dout,
                               const float* dsf, void* dq, void* dk, void* dv, float* dql, float* dkl, float* dld,
                               float* dbeta, float* ds0, float* ws, const int* cu, bool packed, hipStream_t stream) {
    const GdnChunkSizes z = gdn_chunk_sizes(p, packed);
    // the wide areas first: their rows then begin on the cache lines the allocation begins on (64 bytes off, train steps
    // were 6 % slower)
    uint16_t* S = (uint16_t*)ws;
    uint16_t* X = S + 2 * z.state;
    uint16_t* Srest = X + 2 * z.state;
    uint16_t* Xrest = Srest + 2 * z.rest;
    uint16_t* res = Xrest + 2 * z.rest;
    float* du = (float*)(res + 2 * z.wide);
    float* block_ws = du + 2 * z.wide;
    float* gq = block_ws + gdn_pair_workspace_floats(p.B, p.T, p.H, packed);
    float* gk = gq + z.n;
    float* dgq = gk + z.n;
    float* dgk = dgq + z.n;
    float* e = dgk + z.n;
    float* anchor = e + z.n;
    float* ends = anchor + gdn_anchor_count(z.rows) * p.H * chk::kSpanChunks;
    GdnBlockArgs g = {};
    g.q = (const uint16_t*)q; g.k = (const uint16_t*)k; g.v = (const uint16_t*)v; g.dout = (const uint16_t*)dout;
    g.ld = ld; g.beta = beta; g.gq = gq; g.gk = gk; g.s0 = s0; g.dsf = dsf; g.ds0 = ds0;
    g.keep_s = S; g.keep_x = X; g.rest_s = Srest; g.rest_x = Xrest; g.res_rows = res; g.du_rows = du; g.corr = ends;
    g.block_ws = block_ws;
    g.rows = z.rows; g.cu = cu;
    g.B = p.B; g.T = p.T; g.H = p.H; g.dim_k = p.dk; g.dim_v = p.dv;
    chk::GdnArgs c = {};
    c.a.q = g.q; c.a.k = g.k; c.a.v = g.v; c.a.dout = g.dout;
    c.a.dq = (uint16_t*)dq; c.a.dk = (uint16_t*)dk; c.a.dv = (uint16_t*)dv;
    c.a.gq = gq; c.a.gk = gk; c.a.dgq = dgq; c.a.dgk = dgk;
    c.a.B = p.B; c.a.T = p.T; c.a.H = p.H; c.a.cu = cu;
    c.a.nb = p.B; c.a.nh = p.H; c.a.slots = (int)z.slots;
    c.a.nchunk = (p.T + kGdnChunk - 1) / kGdnChunk;
    c.S = S; c.X = X; c.Srest = Srest; c.Xrest = Xrest; c.res = res; c.du = du; c.ld = ld; c.beta = beta; c.e = e; c.anchor = anchor; c.dbeta = dbeta;
    int rc = launch_bwd_gates(ql, kl, gq, gk, z.rows, p.H, stream);
    if (rc == SLA_OK) rc = launch_gdn_block_pair(g, stream);
    if (rc == SLA_OK) rc = p.dk == 64 ? chk::launch_gdn_chunks_dv<64>(c, p.dv, stream) : chk::launch_gdn_chunks_dv<128>(c, p.dv, stream);
    if (rc == SLA_OK) rc = launch_gdn_decay_scan(e, dsf ? ends : nullptr, p.dv / 16, p.B, p.T, p.H, cu, anchor, chk::kSpanChunks, dld, stream);
    if (rc != SLA_OK) return rc;
    return launch_bwd_logits(GateGrad{gq, dgq, 1, 0, dql}, GateGrad{gk, dgk, 1, 0, kl ? dkl : nullptr}, z.rows, p.H, cu, p.B,
                             stream);
}

}  // namespace sla
