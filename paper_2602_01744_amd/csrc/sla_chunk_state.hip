// States at the chunk boundaries (see sla_chunk.h), RetNet and GLA, bf16 tensors:
//     S <- diag(A) S + sum_j (k_j G^K_j p_end / p_j)^T v_j         forward in time; S is kept entering every chunk
//     X <- diag(A) X + sum_t (q_t G^Q_t p_t)^T dout_t              backward in time; X is kept behind every chunk
// with p the decay products from the chunk's start, A = p_end.  No product contracts the state, so it is cut into tiles of
// TK key dimensions x 64 value columns, one workgroup each, whose accumulators (fp32) stay in registers; both directions
// run in one launch.
// Bound by the memory system when there are many sequences and by the chain of chunks when there are few: one barrier per
// chunk, loads two chunks ahead, the decay scan of the next chunk ahead of it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sla.h"
#include "sla_chunk.h"

namespace sla {
namespace chk {

constexpr int kStateThreads = 256;
constexpr int kTileV = 64;

// [64 tokens][units of 8 columns]: both operands of the product are read by columns
__device__ __forceinline__ int state_unit8(int row, int u) { return row * 8 + (u ^ (((row >> 1) << 1) & 6) ^ ((row >> 3) & 1)); }
template <int U>
__device__ __forceinline__ int state_unit(int row, int u) {
    if constexpr (U == 8) return state_unit8(row, u);
    return unit_at<4>(row, u);
}

template <int VAR, int DK, int DV, int TK>
__global__ __launch_bounds__(kStateThreads, 3) void sla_chunk_state_kernel(const Args a) {
    constexpr int NI = TK / 32;           // 16-byte pieces of a key row per lane; key tiles per wave
    constexpr int UK = TK / 8, UV = kTileV / 8;
    constexpr int NTK = DK / TK, NTV = DV / kTileV, NT = NTK * NTV;
    __shared__ __align__(16) uint16_t sk[2][kChunk * TK];
    __shared__ __align__(16) uint16_t sv[2][kChunk * kTileV];
    __shared__ __align__(16) uint16_t sg[VAR == SLA_GLA ? 2 : 1][VAR == SLA_GLA ? kChunk * TK : 8];  // the log decay as loaded
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The tiles of a sequence and head read the same rows: they share an XCD (workgroups are dealt to XCDs round-robin).
    const int place = blockIdx.x >> 3, pair = (place / NT) * 8 + (blockIdx.x & 7), tile = place % NT;
    if (pair >= a.nb * a.nh) return;
    const int b = a.b0 + pair / a.nh, hi = pair % a.nh, h = a.h0 + hi;
    const int kt0 = (tile % NTK) * TK, vt0 = (tile / NTK) * kTileV;
    const bool rev = blockIdx.y != 0;
    const Sequence s = sequence(a, b);
    const int nc = (s.T + kChunk - 1) / kChunk;
    const Rows rx = rows_of<DK>(a, rev ? a.q : a.k, s, b, h);
    const Rows rl = VAR == SLA_GLA ? rows_of<DK>(a, a.ld, s, b, h) : rx;
    const Rows ry = rows_of<DV>(a, rev ? a.dout : a.v, s, b, h);
    const Rows rg = scalars_of(a, rev ? a.gq : a.gk, s, h);
    const float step = VAR == SLA_RETNET ? a.ld_head[h] * kLog2e : 0.f;

    // this wave's accumulators: key tiles ti(i), value columns vt0 + 32 cg ..; D = v^T k: D[value 8g + 4n + e][key tile row r]
    const int wp = TK == 64 ? (w & 1) : 0, cg = w >> 1;
    auto ti = [&](int i) { return TK == 64 ? i : (w & 1); };  // which of the tile pair
    f4 acc[NI][2];
    {
        const float* init = rev ? a.dsf : a.s0;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const int d = kt0 + 32 * wp + key_of(ti(i), r), v = vt0 + 32 * cg + 8 * g + 4 * n;
                acc[i][n] = init ? *(const f4*)(init + (((size_t)b * a.H + h) * DK + d) * DV + v) : f4{0.f, 0.f, 0.f, 0.f};
            }
    }
    struct Pre {
        u4 x[NI], l[NI], y[2];
        float gate;
    };
    // Sums of the log decay along the tokens are a product with a triangle of ones (exact: bf16 values, fp32 sums): column r
    // is token 16 w + r, forward the sum over the tokens behind it, in reverse the sum up to it.
    s8 tri[2], ones;
    {
        u4 x[2], one;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            one[e] = 0x3f803f80u;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int t = 32 * p + 8 * g + 2 * e, me = 16 * w + r;
                const bool lo = rev ? t <= me : t > me, hi2 = rev ? t + 1 <= me : t + 1 > me;
                x[p][e] = (lo ? 0x3f80u : 0u) | (hi2 ? 0x3f800000u : 0u);
            }
        }
        tri[0] = op(x[0]);
        tri[1] = op(x[1]);
        ones = op(one);
    }
    // columns of a staged array (as A operand: its transpose; as B operand: itself), tokens 32 p ..
    auto col_op = [&](const uint16_t* x, int p, int u, int half) {
        const int j = 32 * p + 8 * g + (r >> 2);
        return join(lds_tr(x + 8 * state_unit<UK>(j, u + (r & 3)) + 4 * half), lds_tr(x + 8 * state_unit<UK>(j + 4, u + (r & 3)) + 4 * half));
    };
    const int row = 16 * w + r;  // this lane's token of a chunk; its key columns are kt0 + 32 ii + 8g ..
    auto load = [&](int it, Pre& p) {
        const int t0 = (it >= nc ? nc : rev ? nc - 1 - it : it) * kChunk;  // past the last chunk: zeros
#pragma unroll
        for (int ii = 0; ii < NI; ++ii) {
            if constexpr (VAR == SLA_GLA) p.l[ii] = rl.load(t0 + row, kt0 + 32 * ii + 8 * g);
            p.x[ii] = rx.load(t0 + row, kt0 + 32 * ii + 8 * g);
        }
        p.gate = load_scalar(rg, t0 + row);
#pragma unroll
        for (int n = 0; n < 2; ++n) p.y[n] = ry.load(t0 + (tid >> 3) + 32 * n, vt0 + 8 * (tid & 7));
    };
    auto stage_decay = [&](int it, const Pre& p) {  // a turn ahead of the rest: every wave needs the decay of all tokens
        if constexpr (VAR == SLA_GLA) {
#pragma unroll
            for (int ii = 0; ii < NI; ++ii) *(u4*)(sg[it & 1] + 8 * state_unit<UK>(row, 4 * ii + g)) = p.l[ii];
        }
    };
    auto stage = [&](int it, const Pre& p, float (&A)[NI]) {
        uint16_t* dk = sk[it & 1];
        uint16_t* dv = sv[it & 1];
        const int len = min(kChunk, s.T - (rev ? nc - 1 - it : it) * kChunk);
        float f0 = 0.f, lg = 0.f;
        f4 c[NI][2];
        if constexpr (VAR == SLA_RETNET) {
            f0 = p.gate * ex2(fminf(step * (float)(rev ? row + 1 : len - 1 - row), 0.f));
#pragma unroll
            for (int i = 0; i < NI; ++i) A[i] = ex2(step * (float)len);
        } else {
            lg = __builtin_amdgcn_logf(p.gate);  // log2: the gate multiplies in the exponent
            f4 tot[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) tot[i] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ii = 0; ii < NI; ++ii)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    c[ii][half] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const s8 x = col_op(sg[it & 1], q, 4 * ii, half);
                        mma(c[ii][half], x, tri[q]);
                        if (TK == 64 ? ii == wp : half == (w & 1)) mma(tot[TK == 64 ? half : 0], ones, x);
                    }
                }
#pragma unroll
            for (int i = 0; i < NI; ++i) A[i] = ex2(tot[i][0] * kLog2e);
        }
#pragma unroll
        for (int ii = 0; ii < NI; ++ii) {
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = VAR == SLA_GLA ? ex2(fmaf(c[ii][e >> 2][e & 3], kLog2e, lg)) : f0;
            u4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = pack2(bf_lo(p.x[ii][e]) * f[2 * e], bf_hi(p.x[ii][e]) * f[2 * e + 1]);
            *(u4*)(dk + 8 * state_unit<UK>(row, 4 * ii + g)) = o;
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) *(u4*)(dv + 8 * state_unit<UV>((tid >> 3) + 32 * n, tid & 7)) = p.y[n];
    };
    auto update = [&](int it, const float (&A)[NI]) {
        const int chunk = rev ? nc - 1 - it : it;
        const __amdgpu_buffer_rsrc_t dst = pieces_of<DK, DV>(rev ? a.X : a.S, (size_t)(s.slot0 + chunk) * a.nh + hi);
        // Behind the last token the decay gradient is rowsum(dsf * S_T), with few sums to average a rounding over: the part of
        // it that the state entering the last chunk makes is taken from the states as they are here, in fp32, not from the
        // pieces (T = 8, states in and out: error 2.8e-3 of its norm from those, 1.7e-3 so).
        if (VAR == SLA_GLA && a.end && !rev && it == nc - 1) {
            const size_t bh = (size_t)b * a.H + h;
            const __amdgpu_buffer_rsrc_t x = __builtin_amdgcn_make_buffer_rsrc((void*)(a.dsf + bh * (DK * DV)), 0, DK * DV * 4, kRsrcWord3);
            const __amdgpu_buffer_rsrc_t y = __builtin_amdgcn_make_buffer_rsrc((void*)(a.end + bh * (DK * DV / 32)), 0, DK * DV / 8, kRsrcWord3);
            const int at = 4 * (key_of(0, r) * DV + 8 * g);  // bytes; the second tile of a pair is four rows on
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                float sum = 0.f;
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    const f4 v = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(
                                                            x, at, 4 * ((kt0 + 32 * wp + 4 * ti(i)) * DV + vt0 + 32 * cg + 4 * n), 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum = fmaf(v[e], acc[i][n][e], sum);
                }
                sum = all_groups(sum);
                if (g == 0)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sum), y, 4 * key_of(0, r),
                                                          4 * (((vt0 >> 5) + cg) * DK + kt0 + 32 * wp + 4 * ti(i)), 0);
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            __builtin_amdgcn_raw_buffer_store_b128(pack8(acc[i][0], acc[i][1]), dst,
                                                   16 * lane + piece<DV>((kt0 >> 4) + 2 * wp + ti(i), (vt0 >> 5) + cg), 0, 0);
#pragma unroll
            for (int n = 0; n < 2; ++n) acc[i][n] = acc[i][n] * A[i];
        }
        const uint16_t* dk = sk[it & 1];
        const uint16_t* dv = sv[it & 1];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int j0 = 32 * p + 8 * g + (r >> 2), j1 = j0 + 4;
            s8 fv[2], fk[NI];
#pragma unroll
            for (int n = 0; n < 2; ++n)
                fv[n] = join(lds_tr(dv + 8 * state_unit<UV>(j0, 4 * cg + (r & 3)) + 4 * n),
                             lds_tr(dv + 8 * state_unit<UV>(j1, 4 * cg + (r & 3)) + 4 * n));
#pragma unroll
            for (int i = 0; i < NI; ++i) fk[i] = col_op(dk, p, 4 * wp, ti(i));
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int n = 0; n < 2; ++n) mma(acc[i][n], fv[n], fk[i]);
        }
    };
    if (nc > 0) {
        Pre pa, pb;
        float A[NI];
        load(0, pa);
        load(1, pb);
        stage_decay(0, pa);
        __syncthreads();
        auto turn = [&](int it, Pre& cur, Pre& next) {
            stage(it, cur, A);
            load(it + 2, cur);
            stage_decay(it + 1, next);
            __syncthreads();  // rows of this chunk and the decay of the next are in LDS; the other buffers are free
            update(it, A);
        };
        for (int it = 0; it < nc; it += 2) {
            turn(it, pa, pb);
            if (it + 1 < nc) turn(it + 1, pb, pa);
        }
    }
    if (rev && a.ds0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const int d = kt0 + 32 * wp + key_of(ti(i), r), v = vt0 + 32 * cg + 8 * g + 4 * n;
                *(f4*)(a.ds0 + (((size_t)b * a.H + h) * DK + d) * DV + v) = acc[i][n];
            }
    }
}

template <int VAR, int DK, int DV>
static int launch_tiles(const Args& a, hipStream_t stream) {
    const dim3 block(kStateThreads);
    const unsigned pairs8 = ((unsigned)(a.nb * a.nh) + 7u) / 8u * 8u, dirs = 2;
    if constexpr (DK == 32) {
        hipLaunchKernelGGL((sla_chunk_state_kernel<VAR, DK, DV, 32>), dim3(pairs8 * (DV / kTileV), dirs), block, 0, stream, a);
    } else {
        hipLaunchKernelGGL((sla_chunk_state_kernel<VAR, DK, DV, 64>), dim3(pairs8 * (DK / 64) * (DV / kTileV), dirs), block, 0,
                           stream, a);
    }
    return hipGetLastError() == hipSuccess ? SLA_OK : SLA_ERR_HIP;
}
template <int VAR, int DK>
static int launch_dv(const Args& a, int dv, hipStream_t stream) {
    switch (dv) {
        case 64: return launch_tiles<VAR, DK, 64>(a, stream);
        case 128: return launch_tiles<VAR, DK, 128>(a, stream);
        case 256: return launch_tiles<VAR, DK, 256>(a, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}
template <int VAR>
static int launch_dk(const Args& a, int dk, int dv, hipStream_t stream) {
    switch (dk) {
        case 32: return launch_dv<VAR, 32>(a, dv, stream);
        case 64: return launch_dv<VAR, 64>(a, dv, stream);
        case 128: return launch_dv<VAR, 128>(a, dv, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}
int launch_states(const Args& a, int variant, int dk, int dv, hipStream_t stream) {
    return variant == SLA_GLA ? launch_dk<SLA_GLA>(a, dk, dv, stream) : launch_dk<SLA_RETNET>(a, dk, dv, stream);
}

}  // namespace chk
}  // namespace sla
