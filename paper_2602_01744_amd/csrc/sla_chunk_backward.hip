// Backward pass of RetNet and GLA on bf16 tensors, chunk-parallel (see sla_chunk.h).  One workgroup per 64-token chunk and
// head makes dq, dk, dv, the gate gradients and GLA's decay gradient of the chunk from its rows, the state S entering it
// and the gradient X with respect to the state behind it.  With c_t the running log-decay, a 16-token block as reference:
// p = e^c inside the block, A_b the block's total, qa = q p, kd = k / p, kb = k A / p, and M[t][j] = dout_t . v_j (j <= t):
//     dq'_t = p_t (... ((dout_t S^T) A_0 + N[t][0] kb_0) A_1 + ... + N[t][a] kd_a)        N = M G^K_j, block a of t
//     dk'_j = (A/p_j) (... ((v_j X^T) A_3 + N'[j][3] qa_3) A_2 + ...) + N'[j][b] qa_b / p_j  N' = M^T G^Q_t, block b of j
//     dv'_j = kc_j X + sum_t P[t][j] G^Q_t dout_t       kc = k scaled to the chunk's end, P[t][j] = qa_t . kd_j, or qa . kb
// (the products by A_b run on the fp32 accumulators; every factor but 1/p is <= 1).  RetNet's decay is one number per
// token: it multiplies the 64 x 64 matrices after the products, whatever its size.
//     dq = G^Q dq'  dk = G^K dk'  dv = G^K dv'  dG^Q = q . dq'  dG^K = k . dk'
//     dlog_decay_t = A rowsum(X * S) + sum_j k_j dk_state_j + sum_{s >= t in the chunk} (q_s dq_s - k_s dk_s)
// The first two terms are rowsum(X * S_end), from bf16 operands with fp32 sums, so the decay gradient's error is that of 64
// tokens (T = 2085 128 x 128: 5.3e-3 of its norm against the oracle, the sweeps' 1.6e-2; for the tokens next to the sweeps'
// fp32 anchors 2.8e-3 against 3.8e-3).  In a row's last chunk S and X are taken in fp32 for the first term, see end.
// Against the sweeps of sla_backward.hip, which carry the states through all tokens of a sequence (a call, all launches):
// few sequences 2 to 4 times (B=4 T=500 H=8 128 x 128 GLA 109 -> 45 us; B=8 T=4096 H=4 128 x 256 GLA 514, in four segments,
// -> 312 us), B=8 T=2048 H=16 128 x 128 GLA 406 -> 393 us, RetNet 300 -> 282 us: there the memory system bounds it, 0.84 GB in
// and 0.31 GB out in 221 us (GLA).  Small batches are bound by one workgroup's own latency, 19 us.  Which calls it takes:
// backward_chunks_take() in sla_chunk_plan.h.
#include <hip/hip_runtime.h>
#include <stdint.h>


#include "sla.h"
#include "sla_chunk.h"
#include "sla_chunk_plan.h"
#include "sla_gate_grad.h"

namespace sla {

int launch_bwd_gates(const float* ql, const float* kl, float* gq, float* gk, size_t rows, int H, hipStream_t stream);

namespace chk {

int launch_states(const Args& a, int variant, int dk, int dv, hipStream_t stream);

constexpr int kThreads = 256;

// Four waves.  For dq and dk a wave takes 32 key dimensions and TB = DK / 32 of the four token blocks, for dv and P one
// token block.  LDS, in bytes; 80 KB at most, so that two workgroups share a compute unit and one's loads run under the
// other's products.
template <int VAR, int DK>
struct Lds {
    static constexpr int WD = DK / 32, WT = 4 / WD, TB = WD;
    static constexpr int rows = kChunk * DK * 2;
    static constexpr int oQ = 0;                              // qa (RetNet: q)
    static constexpr int oK = oQ + rows;                      // kd (RetNet: k)
    static constexpr int oKB = oK + rows;                     // kb (GLA)
    static constexpr int oV = VAR == SLA_GLA ? oKB + rows : oKB;  // v, dout, X: 32 value columns at a time
    static constexpr int oDO = oV + kChunk * 64;
    static constexpr int oX = oDO + kChunk * 64;
    static constexpr int matrix = kChunk * kChunk * 2;
    static constexpr int oN = oV, oN2 = oN + matrix;          // after the value columns: N, N'
    static constexpr int oKC = oV;                            // before them: k scaled to the chunk's end (GLA)
    static constexpr int shared = (oX + DK * 64 > oN2 + matrix ? oX + DK * 64 : oN2 + matrix);
    static constexpr int oA = (shared > oKC + rows ? shared : oKC + rows);  // GLA: A_b [4][DK]
    static constexpr int oGate = VAR == SLA_GLA ? oA + 4 * DK * 4 : oA;     // gates [2][64]
    static constexpr int oCorr = oGate + 2 * kChunk * 4;      // GLA: rowsum(X * S) [DK]
    static constexpr int oFin = oCorr + DK * 4;               // GLA, WT > 1: the waves' sums of k dk_state [WT][DK]
    static constexpr int oDec = oFin + (WT > 1 ? WT * DK * 4 : 0);  // ... and of q dq - k dk [WT][DK]
    static constexpr int oQ32 = oDec + (WT > 1 ? WT * DK * 4 : 0);  // GLA: qa of block 3 and kb of block 0 scaled to the middle
    static constexpr int oK32 = oQ32 + 16 * DK * 2;
    static constexpr int oScan = oK32 + 16 * DK * 2;          // GLA: 16 x 32 decay steps per wave
    static constexpr int total = VAR != SLA_GLA ? oCorr : oScan + 4 * 1024;
    static constexpr int oRed = oQ;                           // at the end: partial gate gradients [2][WD][64]
    static_assert(total <= 80 * 1024, "two workgroups per compute unit");
};

template <int VAR, int DK, int DV>
__global__ __launch_bounds__(kThreads, 2) void sla_chunk_backward_kernel(const Args a) {
    typedef Lds<VAR, DK> L;
    constexpr bool GLA = VAR == SLA_GLA;
    // GLA at width 128: q, k and the decay are loaded a second time for the last part; kept, they would spill (this
    // launch, B=8 T=2048 H=16: 291 us against 260 when the choice was made, 221 now)
    constexpr bool kReload = GLA && DK == 128;
    constexpr int WD = L::WD, WT = L::WT, TB = L::TB, U = DK / 8, NS = DV / 32, NM = 3;
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t* sq = (uint16_t*)(smem + L::oQ);
    uint16_t* sk = (uint16_t*)(smem + L::oK);
    uint16_t* skb = (uint16_t*)(smem + L::oKB);
    uint16_t* sv = (uint16_t*)(smem + L::oV);
    uint16_t* sdo = (uint16_t*)(smem + L::oDO);
    uint16_t* sx = (uint16_t*)(smem + L::oX);
    uint16_t* sn = (uint16_t*)(smem + L::oN);
    uint16_t* sn2 = (uint16_t*)(smem + L::oN2);
    float* sA = (float*)(smem + L::oA);
    float* sgq = (float*)(smem + L::oGate);
    float* sgk = sgq + kChunk;
    float* scorr = (float*)(smem + L::oCorr);
    float* sfin = (float*)(smem + L::oFin);
    float* sdec = (float*)(smem + L::oDec);
    float* sred = (float*)(smem + L::oRed);
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wd = w % WD, wt = w / WD;

    // Chunk and head.  The heads of a chunk are neighbours, and every XCD gets a contiguous range: their gates share lines.
    const int per = (int)(gridDim.x >> 3), id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (id >= a.slots * a.nh) return;
    const int hi = id % a.nh, slot = id / a.nh, h = a.h0 + hi;
    int b, chunk;
    if (!chunk_of(a, slot, b, chunk)) return;
    const Sequence s = sequence(a, b);
    const int t0 = chunk * kChunk, len = min(kChunk, s.T - t0);
    const size_t state = (size_t)slot * a.nh + hi;
    const __amdgpu_buffer_rsrc_t rS = pieces_of<DK, DV>(a.S, state), rX = pieces_of<DK, DV>(a.X, state);
    const Rows rq = rows_of<DK>(a, a.q, s, b, h), rk = rows_of<DK>(a, a.k, s, b, h);
    const Rows rl = GLA ? rows_of<DK>(a, a.ld, s, b, h) : rq;
    const Rows rv = rows_of<DV>(a, a.v, s, b, h), rdo = rows_of<DV>(a, a.dout, s, b, h);
    const float step = GLA ? 0.f : a.ld_head[h] * kLog2e;
    const int d0 = 32 * wd + 8 * g, m0 = TB * wt;  // this lane's eight key dimensions; its tokens 16 m + r, m0 <= m < m0 + TB

    // v and dout: 64 tokens x 4 units of 8 columns per step of 32 columns, loaded for two steps at once (whole 128-byte
    // lines); S and X pieces of the wave's two key tiles
    struct Pre {
        u4 v[2], o[2], S[2], X[2];
    } pre;
    auto load_rows = [&](int c) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            pre.v[i] = rv.load(t0 + (tid >> 2), 32 * (c + i) + 8 * (tid & 3));
            pre.o[i] = rdo.load(t0 + (tid >> 2), 32 * (c + i) + 8 * (tid & 3));
        }
    };
    auto load_states = [&](int c) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            pre.S[i] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rS, 16 * lane + piece<DV>(2 * wd + i, c), 0, 2));
            pre.X[i] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rX, 16 * lane + piece<DV>(2 * wd + i, c), 0, 2));
        }
    };
    u4 qx[TB], kx[TB], lx[TB];
    auto load_key = [&](int m) {
        const int t = t0 + 16 * (m0 + m) + r;
        if constexpr (GLA) lx[m] = rl.load(t, d0);
        kx[m] = rk.load(t, d0);
    };
    auto load_query = [&](int m) { qx[m] = rq.load(t0 + 16 * (m0 + m) + r, d0); };
#pragma unroll
    for (int m = TB - 1; m >= 0; --m) {
        load_key(m);
        load_query(m);
    }
    u4 ll[4];  // decay of the other waves' blocks
    if constexpr (GLA && WT > 1) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (m < m0 || m >= m0 + TB) ll[m] = rl.load(t0 + 16 * m + r, d0);
    }
    if (tid < kChunk) {
        sgq[tid] = load_scalar(scalars_of(a, a.gq, s, h), t0 + tid);
        sgk[tid] = load_scalar(scalars_of(a, a.gk, s, h), t0 + tid);
    }
    if (GLA && a.end && t0 + kChunk >= s.T && tid < DK) {  // the row's end: rowsum(X * S) from the state kernel, in fp32
        const float* src = a.end + ((size_t)b * a.H + h) * (DV / 32) * DK + tid;
        float sum = 0.f;
#pragma unroll
        for (int n = 0; n < DV / 32; ++n) sum += src[n * DK];
        scorr[tid] = sum;
    }
    load_rows(0);
    load_states(0);

    // Sums of a block's log2 decay along its tokens, in this lane's layout: a product with a triangle of ones (exact: bf16
    // values, fp32 sums) through a scratch tile of the wave.  c[e]: up to token r; with `ones` the block's total.
    uint16_t* scr = (uint16_t*)(smem + L::oScan) + 512 * w;
    s8 tri, ones;
    {
        u4 x, y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = 8 * g + 2 * e;
            x[e] = (j <= r ? 0x3f80u : 0u) | (j + 1 <= r ? 0x3f800000u : 0u);
            y[e] = g < 2 ? 0x3f803f80u : 0u;
        }
        tri = op(x);
        if (g >= 2) tri = op(u4{0u, 0u, 0u, 0u});
        ones = op(y);
    }
    auto scan = [&](const u4& l, const s8& with, float* c) {
        *(u4*)(scr + 8 * unit_at<4>(r, g)) = l;
        const int row = 8 * (g & 1) + (r >> 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f4 x = {0.f, 0.f, 0.f, 0.f};
            mma(x, join(lds_tr(scr + 8 * unit_at<4>(row, r & 3) + 4 * i), lds_tr(scr + 8 * unit_at<4>(row + 4, r & 3) + 4 * i)), with);
#pragma unroll
            for (int e = 0; e < 4; ++e) c[4 * i + e] = x[e] * kLog2e;
        }
    };
    if constexpr (GLA) {
        float A[4][8], later[8];
        if constexpr (WT > 1) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (m < m0 || m >= m0 + TB) {
                    scan(ll[m], ones, A[m]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) A[m][e] = ex2(A[m][e]);
                }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) later[e] = 1.f;
#pragma unroll
        for (int m = 3; m >= 0; --m) {
            if (WT > 1 && (m < m0 || m >= m0 + TB)) {
                if (m > m0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) later[e] *= A[m][e];
                }
                continue;
            }
            const int mm = WT == 1 ? m : m % TB;
            float c[8], f[6][8];
            scan(lx[mm], tri, c);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float q = bf_at(qx[mm], e), k = bf_at(kx[mm], e), p = ex2(c[e]);
                A[m][e] = row_last(p);
                f[0][e] = q * p;
                f[1][e] = k * ex2(-c[e]);
                f[2][e] = f[1][e] * A[m][e];
                f[3][e] = f[2][e] * later[e];
                later[e] *= A[m][e];
            }
            auto put = [&](int offset, int row, const float* x) {
                *(u4*)((uint16_t*)(smem + offset) + 8 * unit_at<U>(row, 4 * wd + g)) =
                    u4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7])};
            };
            put(L::oQ, 16 * m + r, f[0]);
            put(L::oK, 16 * m + r, f[1]);
            put(L::oKB, 16 * m + r, f[2]);
            put(L::oKC, 16 * m + r, f[3]);
            if (m == 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[4][e] = f[2][e] * A[1][e];
                put(L::oK32, r, f[4]);
            }
            if (m == 3 && WT == 4) {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[5][e] = f[0][e] * A[2][e];
                put(L::oQ32, r, f[5]);
            }
            if (m == 2 && WT < 4) {  // block 3's rows are in registers still
                constexpr int kLast = TB - 1;
                float c3[8];
                scan(lx[kLast], tri, c3);
#pragma unroll
                for (int e = 0; e < 8; ++e) f[5][e] = bf_at(qx[kLast], e) * ex2(c3[e]) * A[2][e];
                put(L::oQ32, r, f[5]);
            }
            if (r == 0) {
                *(f4*)(sA + m * DK + d0) = f4{A[m][0], A[m][1], A[m][2], A[m][3]};
                *(f4*)(sA + m * DK + d0 + 4) = f4{A[m][4], A[m][5], A[m][6], A[m][7]};
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int m = 0; m < TB; ++m) {
            const int at = 8 * unit_at<U>(16 * (m0 + m) + r, 4 * wd + g);
            *(u4*)(sq + at) = qx[m];
            *(u4*)(sk + at) = kx[m];
        }
    }
    __syncthreads();

    // P of the wave's token block (columns j), as the B operand whose slots (half, g, e) are t = 16 half + 4g + e, and kc_j
    const int jb = w, j = 16 * jb + r;
    s8 fp[2], fkc[DK / 32];
    auto row_op = [&](const uint16_t* x, int row, int c) { return op(*(const u4*)(x + 8 * unit_at<U>(row, 4 * c + g))); };
    {
        f4 P[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) P[m] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < DK / 32; ++c) fkc[c] = row_op(GLA ? (const uint16_t*)(smem + L::oKC) : sk, j, c);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (m < jb) continue;
            const uint16_t* xq = sq;
            const uint16_t* xk = sk;
            int tq = 16 * m + r, tk = j;
            if constexpr (GLA) {  // the reference of the pair: block jb's start, its end (adjacent blocks) or the chunk's middle
                if (m > jb) xk = skb;
                if (m >= 2 && jb == 0) xk = (const uint16_t*)(smem + L::oK32), tk = r;
                if (m == 3 && jb <= 1) xq = (const uint16_t*)(smem + L::oQ32), tq = r;
            }
#pragma unroll
            for (int c = 0; c < DK / 32; ++c) mma(P[m], row_op(xq, tq, c), row_op(xk, tk, c));
            const f4 gate = *(const f4*)(sgq + 16 * m + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = 16 * m + 4 * g + e;
                float x = P[m][e] * gate[e];
                if constexpr (!GLA) x *= ex2(step * (float)max(t - j, 0));
                P[m][e] = t >= j ? x : 0.f;
            }
        }
        fp[0] = op(pack8(P[0], P[1]));
        fp[1] = op(pack8(P[2], P[3]));
    }

    // ---- the value columns, 32 at a time: M, dout S^T, v X^T, and dv
    f4 aq[TB][2], ak[TB][2], M[NM];
#pragma unroll
    for (int m = 0; m < TB; ++m)
#pragma unroll
        for (int i = 0; i < 2; ++i) aq[m][i] = ak[m][i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < NM; ++x) M[x] = f4{0.f, 0.f, 0.f, 0.f};
    f4 corr[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};  // GLA: S X^T of a key tile; its diagonal is wanted
    for (int c2 = 0; c2 < NS; c2 += 2)
#pragma unroll
    for (int x2 = 0; x2 < 2; ++x2) {
        const int c = c2 + x2;
        __syncthreads();  // the readers of what lies here are done
        s8 fS[2], fX[2];
        *(u4*)(sv + 8 * unit_at<4>(tid >> 2, tid & 3)) = pre.v[x2];
        *(u4*)(sdo + 8 * unit_at<4>(tid >> 2, tid & 3)) = pre.o[x2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            fS[i] = op(pre.S[i]);
            fX[i] = op(pre.X[i]);
            const int row = 32 * wd + key_of(i, r);
            if (wt == 0) *(u4*)(sx + 8 * (row * 4 + (g ^ ((row >> 3) & 3)))) = pre.X[i];
            if constexpr (GLA) mma(corr[i], fS[i], fX[i]);
        }
        if (x2 == 1 && c + 1 < NS) load_rows(c + 1);
        if (c + 1 < NS) load_states(c + 1);
        __syncthreads();
        auto slab = [&](const uint16_t* x, int row) { return op(*(const u4*)(x + 8 * unit_at<4>(row, g))); };
#pragma unroll
        for (int m = 0; m < TB; ++m) {
            const s8 fo = slab(sdo, 16 * (m0 + m) + r), fv = slab(sv, 16 * (m0 + m) + r);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                mma(aq[m][i], fS[i], fo);
                mma(ak[m][i], fX[i], fv);
            }
        }
#pragma unroll
        for (int x = 0; x < NM; ++x) {
            const int tile = w + 4 * x;
            if (tile < 10) {
                const s8 fo = slab(sdo, 16 * (int)((kTileT >> (4 * tile)) & 15) + r);
                const s8 fv = slab(sv, 16 * (int)((kTileJ >> (4 * tile)) & 15) + r);
                mma(M[x], fo, fv);
            }
        }
        {
            f4 y[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int d = 0; d < DK / 32; ++d) {
                const int row = 32 * d + 8 * g + (r >> 2);
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const uint16_t* p0 = sx + 8 * (row * 4 + ((r & 3) ^ ((row >> 3) & 3))) + 4 * x;
                    mma(y[x], join(lds_tr(p0), lds_tr(p0 + 4 * 32)), fkc[d]);  // row + 4: the same swizzle
                }
            }
            if constexpr (!GLA) {
                const float f = ex2(fminf(step * (float)(len - 1 - j), 0.f));
                y[0] = y[0] * f;
                y[1] = y[1] * f;
            }
#pragma unroll
            for (int pp = 0; pp < 2; ++pp) {
                if (pp == 0 && jb >= 2) continue;
                const int row = 32 * pp + 4 * g + (r >> 2);
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    mma(y[x], join(lds_tr(sdo + 8 * unit_at<4>(row, r & 3) + 4 * x), lds_tr(sdo + 8 * unit_at<4>(row + 16, r & 3) + 4 * x)),
                        fp[pp]);
            }
            const float gk = sgk[j];
            rows_of<DV>(a, a.dv, s, b, h).put(t0 + j, 32 * c + 8 * g, pack8(y[0] * gk, y[1] * gk));
        }
    }
    __syncthreads();

    // ---- N[t][j] and N'[j][t]; meanwhile the rows of k and the decay come back where registers did not keep them
    if constexpr (kReload) {
#pragma unroll
        for (int m = TB - 1; m >= (TB > 2 ? TB - 2 : 0); --m) load_key(m);
    }
    auto n_at = [&](uint16_t* x, int row, int col) { return x + 8 * unit_at<8>(row, col >> 3) + (col & 7); };
#pragma unroll
    for (int x = 0; x < NM; ++x) {
        const int tile = w + 4 * x;
        if (tile < 10) {
            const int tb = 16 * (int)((kTileT >> (4 * tile)) & 15), jb = 16 * (int)((kTileJ >> (4 * tile)) & 15);
            const f4 gq = *(const f4*)(sgq + tb + 4 * g);
            const float gk = sgk[jb + r];
            f4 n2;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = tb + 4 * g + e, j = jb + r;
                float y = M[x][e];
                if constexpr (!GLA) y *= ex2(step * (float)max(t - j, 0));
                if (x == 0) y = t >= j ? y : 0.f;  // the first four tiles are the diagonal's
                n2[e] = y * gq[e];
                *n_at(sn, t, j) = (uint16_t)pack2(y * gk, 0.f);
            }
            *(u2*)n_at(sn2, jb + r, tb + 4 * g) = pack4(n2);
        }
    }
    if constexpr (!GLA) {  // the products below take 32 tokens at a time: the tiles above the diagonal inside them
        for (int x = tid; x < 128; x += kThreads) {
            const int blk = x >> 6, row = (x & 63) >> 2, col = 4 * (x & 3);
            *(u2*)n_at(sn, 32 * blk + row, 32 * blk + 16 + col) = u2{0u, 0u};
            *(u2*)n_at(sn2, 32 * blk + 16 + row, 32 * blk + col) = u2{0u, 0u};
        }
    }
    if (GLA && !(a.end && t0 + kChunk >= s.T)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float lo = (r & 1) ? corr[i][1] : corr[i][0], hi2 = (r & 1) ? corr[i][3] : corr[i][2];
            if (g == (r >> 2) && wt == 0) scorr[32 * wd + key_of(i, r)] = (r & 2) ? hi2 : lo;
        }
    }
    __syncthreads();

    // ---- dq, dk of the wave's 32 dimensions.  Columns of a [token][DK] array: slots 8g .. 8g + 7 are rows `row0` ..
    auto col_op = [&](const uint16_t* x, int row0, int i) {
        const int row = row0 + (r >> 2);
        return join(lds_tr(x + 8 * unit_at<U>(row, 4 * wd + (r & 3)) + 4 * i), lds_tr(x + 8 * unit_at<U>(row + 4, 4 * wd + (r & 3)) + 4 * i));
    };
    auto n_op = [&](uint16_t* x, int row, int col) { return op(*(const u4*)n_at(x, row, col)); };
    auto n_half = [&](uint16_t* x, int row, int col) {  // 16 slots of one block, the others zero
        const u4 v = *(const u4*)n_at(x, row, col + 8 * (g & 1));
        return op(g < 2 ? v : u4{0u, 0u, 0u, 0u});
    };
    auto put_row = [&](uint16_t* x, int t, const float* y) {
        rows_of<DK>(a, x, s, b, h).put(t0 + t, d0, pack8(f4{y[0], y[1], y[2], y[3]}, f4{y[4], y[5], y[6], y[7]}));
    };
    auto decay = [&](f4* x, int blk) {
        x[0] = x[0] * *(const f4*)(sA + blk * DK + d0);
        x[1] = x[1] * *(const f4*)(sA + blk * DK + d0 + 4);
    };
    // GLA: what holds for the whole chunk in dlog_decay, A rowsum(X S) + sum k dk_state; decay from a block's end to the chunk's
    float fin[8], later[8];
    if constexpr (GLA) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            fin[e] = 0.f;
            later[e] = 1.f;
#pragma unroll
            for (int m = TB; m < 4; ++m)
                if (m >= m0 + TB) later[e] *= sA[m * DK + d0 + e];
        }
    }
    float dgk[TB], dgq[TB];
#pragma unroll
    for (int mm = TB - 1; mm >= 0; --mm) {  // dk; ak[mm] becomes k dk
        const int m = m0 + mm, t = 16 * m + r;
        if (kReload && mm >= 2) load_key(mm - 2);
        if (kReload && mm < 2) load_query(TB > 1 ? TB - 2 + mm : 0);
        const float gk = sgk[t];
        f4 k2[2] = {ak[mm][0], ak[mm][1]}, kd2[2];
        float yk[8];
        if constexpr (GLA) {
            // the blocks behind m from the last one down; block m apart
#pragma unroll
            for (int bk = 3; bk > 0; --bk) {
                if (bk <= m) continue;
                const s8 n = n_half(sn2, t, 16 * bk);
                decay(k2, bk);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(k2[i], col_op(sq, 16 * bk + 8 * (g & 1), i), n);
            }
            const s8 n = n_half(sn2, t, 16 * m);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                kd2[i] = f4{0.f, 0.f, 0.f, 0.f};
                mma(kd2[i], col_op(sq, 16 * m + 8 * (g & 1), i), n);
            }
            float c[8];
            scan(lx[mm], tri, c);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float ip = ex2(-c[e]), A = row_last(ex2(c[e])), k = bf_at(kx[mm], e);
                yk[e] = ip * (A * k2[e >> 2][e & 3] + kd2[e >> 2][e & 3]);
                fin[e] = fmaf(ak[mm][e >> 2][e & 3] * gk, k * (ip * A * later[e]), fin[e]);
                later[e] *= A;
            }
        } else {
            const float fk = ex2(fminf(step * (float)(len - 1 - t), 0.f));
#pragma unroll
            for (int i = 0; i < 2; ++i) k2[i] = k2[i] * fk;
#pragma unroll
            for (int pp = 0; pp < 2; ++pp) {
                if (32 * pp + 16 < 16 * m) continue;
                const s8 n = n_op(sn2, t, 32 * pp + 8 * g);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(k2[i], col_op(sq, 32 * pp + 8 * g, i), n);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) yk[e] = k2[e >> 2][e & 3];
        }
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float k = bf_at(kx[mm], e);
            sum = fmaf(k, yk[e], sum);
            yk[e] *= gk;
            if constexpr (GLA) ak[mm][e >> 2][e & 3] = k * yk[e];
        }
        dgk[mm] = all_groups(sum);
        put_row(a.dk, t, yk);
        __builtin_amdgcn_sched_barrier(0);  // one block at a time: the registers do not hold two
    }
    if constexpr (GLA) {
#pragma unroll
        for (int e = 0; e < 8; ++e) fin[e] = row_all(fin[e]);
        if constexpr (WT > 1) {
            if (r == 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) sfin[wt * DK + d0 + e] = fin[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) fin[e] = fmaf(scorr[d0 + e], later[e], fin[e]);
        }
    }
    float dec[8], dl[WT > 1 ? TB : 1][8];  // GLA: sums of q dq - k dk over the wave's later blocks; dlog_decay, not whole yet
#pragma unroll
    for (int e = 0; e < 8; ++e) dec[e] = 0.f;
#pragma unroll
    for (int mm = TB - 1; mm >= 0; --mm) {  // dq and the decay
        const int m = m0 + mm, t = 16 * m + r;
        if (kReload && mm >= 2) load_query(mm - 2);
        const float gq = sgq[t];
        f4 q2[2] = {aq[mm][0], aq[mm][1]};
        float yq[8], sum = 0.f;
        if constexpr (GLA) {
            // the blocks before m - 1 one by one, then m - 1 (through kb) and m (through kd) in one product
#pragma unroll
            for (int bk = 0; bk < 2; ++bk) {
                if (bk + 1 >= m) continue;
                const s8 n = n_half(sn, t, 16 * bk);
                decay(q2, bk);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(q2[i], col_op(skb, 16 * bk + 8 * (g & 1), i), n);
            }
            if (m > 0) {
                decay(q2, m - 1);
                const s8 n = n_op(sn, t, 16 * (m - 1) + 8 * g);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(q2[i], col_op(g < 2 ? skb : sk, 16 * (m - 1) + 8 * g, i), n);
            } else {
                const s8 n = n_half(sn, t, 0);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(q2[i], col_op(sk, 8 * (g & 1), i), n);
            }
            float c[8];
            scan(lx[mm], tri, c);
#pragma unroll
            for (int e = 0; e < 8; ++e) yq[e] = ex2(c[e]) * q2[e >> 2][e & 3];
        } else {
            const float fq = ex2(step * (float)(t + 1));
#pragma unroll
            for (int i = 0; i < 2; ++i) q2[i] = q2[i] * fq;
#pragma unroll
            for (int pp = 0; pp < 2; ++pp) {
                if (32 * pp > 16 * m) continue;
                const s8 n = n_op(sn, t, 32 * pp + 8 * g);
#pragma unroll
                for (int i = 0; i < 2; ++i) mma(q2[i], col_op(sk, 32 * pp + 8 * g, i), n);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) yq[e] = q2[e >> 2][e & 3];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float q = bf_at(qx[mm], e);
            sum = fmaf(q, yq[e], sum);
            yq[e] *= gq;
            if constexpr (GLA) {
                const float x = row_suffix(fmaf(q, yq[e], -ak[mm][e >> 2][e & 3]));
                dl[WT > 1 ? mm : 0][e] = dec[e] + x + (WT > 1 ? 0.f : fin[e]);
                dec[e] += row_first(x);
            }
        }
        dgq[mm] = all_groups(sum);
        put_row(a.dq, t, yq);
        if constexpr (GLA && WT == 1) put_row(a.dld, t, dl[0]);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (GLA && WT > 1) {
        if (r == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sdec[wt * DK + d0 + e] = dec[e];
        }
    }
    __syncthreads();
    if constexpr (GLA && WT > 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float x = 0.f, A = 1.f;
#pragma unroll
            for (int n = 0; n < WT; ++n) x += sfin[n * DK + d0 + e] + (n > wt ? sdec[n * DK + d0 + e] : 0.f);
#pragma unroll
            for (int m = 0; m < 4; ++m) A *= sA[m * DK + d0 + e];
            x = fmaf(scorr[d0 + e], A, x);
#pragma unroll
            for (int mm = 0; mm < TB; ++mm) dl[mm][e] += x;
        }
#pragma unroll
        for (int mm = 0; mm < TB; ++mm) put_row(a.dld, 16 * (m0 + mm) + r, dl[mm]);
    }
    if (g == 0) {
#pragma unroll
        for (int mm = 0; mm < TB; ++mm) {
            sred[wd * kChunk + 16 * (m0 + mm) + r] = dgq[mm];
            sred[(WD + wd) * kChunk + 16 * (m0 + mm) + r] = dgk[mm];
        }
    }
    __syncthreads();
    for (int i = tid; i < 2 * kChunk; i += kThreads) {
        const int t = i & (kChunk - 1), which = i / kChunk;
        if (t < len) {
            float x = 0.f;
#pragma unroll
            for (int n = 0; n < WD; ++n) x += sred[(which * WD + n) * kChunk + t];
            (which ? a.dgk : a.dgq)[(s.tok0 + t0 + t) * a.H + h] = x;
        }
    }
}

template <int VAR, int DK, int DV>
static int launch_chunks(const Args& a, hipStream_t stream) {
    typedef Lds<VAR, DK> L;
    if (!allow_lds<sla_chunk_backward_kernel<VAR, DK, DV>>(L::total)) return SLA_ERR_HIP;
    const unsigned n = ((unsigned)a.slots * a.nh + 7u) / 8u * 8u;
    hipLaunchKernelGGL((sla_chunk_backward_kernel<VAR, DK, DV>), dim3(n), dim3(kThreads), (size_t)L::total, stream, a);
    return hipGetLastError() == hipSuccess ? SLA_OK : SLA_ERR_HIP;
}
template <int VAR, int DK>
static int launch_chunks_dv(const Args& a, int dv, hipStream_t stream) {
    switch (dv) {
        case 64: return launch_chunks<VAR, DK, 64>(a, stream);
        case 128: return launch_chunks<VAR, DK, 128>(a, stream);
        case 256: return launch_chunks<VAR, DK, 256>(a, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}

template <int VAR>
static int launch_chunks_dk(const Args& a, int dk, int dv, hipStream_t stream) {
    switch (dk) {
        case 32: return launch_chunks_dv<VAR, 32>(a, dv, stream);
        case 64: return launch_chunks_dv<VAR, 64>(a, dv, stream);
        case 128: return launch_chunks_dv<VAR, 128>(a, dv, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}

}  // namespace chk

int launch_backward_chunks(const sla_params& p, const void* q, const void* k, const void* v, const float* ql,
                           const float* kl, const void* ld, const float* s0, const void* dout, const float* dsf, void* dq,
                           void* dk, void* dv, float* dql, float* dkl, void* dld, float* ds0, float* ws, size_t floats,
                           const int* cu, bool packed, hipStream_t stream) {
    const size_t rows = packed ? (size_t)p.T : (size_t)p.B * p.T, n = chunk_round4(rows * p.H);
    chk::Args a = {};
    a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.dout = (const uint16_t*)dout;
    a.ld = p.variant == SLA_GLA ? (const uint16_t*)ld : nullptr;
    a.ld_head = p.variant == SLA_RETNET ? (const float*)ld : nullptr;
    a.s0 = s0; a.dsf = dsf; a.ds0 = ds0;
    a.dq = (uint16_t*)dq; a.dk = (uint16_t*)dk; a.dv = (uint16_t*)dv; a.dld = (uint16_t*)dld;
    const ChunkParts parts = backward_chunks_parts(p, packed, floats);
    a.S = (chk::u4*)ws;  // the states first: on the cache lines that the allocation begins on
    a.X = (chk::u4*)(ws + parts.floats / 2);
    float *gq = ws + parts.floats, *gk = gq + n;
    a.gq = gq; a.gk = gk; a.dgq = gk + n; a.dgk = gk + 2 * n;
    a.end = p.variant == SLA_GLA && dsf ? gk + 3 * n : nullptr;  // n floats each: q's and k's gates and their gradients
    a.B = p.B; a.T = p.T; a.H = p.H; a.cu = cu;
    a.head_major = (p.flags & SLA_FLAG_HEAD_MAJOR) != 0;
    a.nchunk = (p.T + chk::kChunk - 1) / chk::kChunk;
    int rc = launch_bwd_gates(ql, kl, gq, gk, rows, p.H, stream);
    for (int b = 0; b < p.B && rc == SLA_OK; b += parts.nb)
        for (int h = 0; h < p.H && rc == SLA_OK; h += parts.nh) {
            a.b0 = b; a.nb = std::min(parts.nb, p.B - b);
            a.h0 = h; a.nh = std::min(parts.nh, p.H - h);
            a.slots = packed ? parts.slots : a.nb * a.nchunk;
            rc = chk::launch_states(a, p.variant, p.dk, p.dv, stream);
            if (rc == SLA_OK)
                rc = p.variant == SLA_GLA ? chk::launch_chunks_dk<SLA_GLA>(a, p.dk, p.dv, stream)
                                          : chk::launch_chunks_dk<SLA_RETNET>(a, p.dk, p.dv, stream);
        }
    if (rc != SLA_OK) return rc;
    return launch_bwd_logits(GateGrad{gq, a.dgq, 1, 0, dql}, GateGrad{gk, a.dgk, 1, 0, kl ? dkl : nullptr}, rows, p.H, cu,
                             p.B, stream);
}

}  // namespace sla
