// SLA recurrent decode step for gfx950 (MI355X): Eq. 5-6 with the Sec. 5.1 recurrences for ONE token per
// (batch, head), the constant-memory inference form (Sec. 3.2, Recurrent Implementation; derived in Appendix A).
//
// The step reads and rewrites the whole state, 2 * dk * dv * 4 bytes per head against O(dk * dv) flops: it is
// HBM-bound, so the kernel is a streaming read-modify-write.  A workgroup of 256 threads owns DS adjacent value
// columns of one (batch, head): no step of the recurrence mixes value columns, so the slices are independent.
// Thread (rg, c4) owns four adjacent columns of the rows rg, rg + NRG, rg + 2 NRG, ...; every load of the workgroup
// (logits or projection, q, k, decay, v, then the state) is issued in the order of use before anything waits, and the
// state stays in registers between the read and the write -- also for the delta rule, whose write depends on a
// reduction (k S) over the whole slice.  Sums over rows meet by shuffles inside a wave and through LDS between the four
// waves.  The slices of a head run on one XCD.
// Slice width: 64 columns (8 state rows per thread at dk = 128).  32 while 64 give at most 2 dk workgroups: the call is
// then one round of loads and stores whose length is the rows per thread (64 / 32 columns, us: B=2 H=64 128 x 64
// 3.8 / 3.5, B=2 H=32 64 x 64 3.1 / 3.0, but B=8 H=32 64 x 64 3.5 / 3.6); from there on 32 pays for twice the q, k, decay
// and gate loads, and 128 and more have fewer wavefronts per compute unit (B=64 H=16 128 x 256 49.9 / 52.4).
// With the projection fused every slice forms all H logits again, so 32 end at dk workgroups (B=8 H=16 128 x 128
// 5.1 / 5.3; B=16 H=16 32 x 64 3.6 / 3.9), and past 256 slices are eight state rows per thread wide (against 64 columns,
// GLA: B=64 H=64 32 x 256 48 -> 42, B=8 H=64 64 x 128 8.4 -> 8.1, B=8 H=64 32 x 256 9.3 -> 7.2), for GLA sixteen
// beyond 32 heads and 512 workgroups (B=16 H=48 128 x 128 20.1 -> 17.2, B=4 H=64 128 x 256 12.8 -> 11.8; B=4 H=64 128 x 128
// 8.3 -> 8.8; the delta rule, whose k S waits for the whole slice, B=16 H=64 128 x 128 26.9 -> 28.7).
// Kernel time in us against one workgroup per (batch, head) and the gates' loads behind the state's, the earlier form
// (bf16, graph of 48 steps; "far": over several states, so that they come from HBM, "near": one state, which the
// memory-side cache holds):
//     B   H  dk x dv                      near           far
//     1   4  128 x 256 GLA, fused      6.2 ->  3.6
//     8   16 128 x 128 GLA             5.4 ->  4.5    6.4 ->  4.8
//     32  16 128 x 128 GLA             9.5 ->  8.9   16.2 -> 15.8
//     64  16 128 x 128 delta rule     23.0 -> 21.7   30.9 -> 28.2 (4.8 TB/s)
//     64  16 128 x 128 GLA, fused     21.7 -> 22.4   29.7 -> 29.3
//     64  16 128 x 256 GLA            48.9 -> 40.7   61.8 -> 50.3 (5.3 TB/s)
//     16  64 128 x 256 GLA, fused     57.4 -> 48.1   68.8 -> 63.1
//     64  64 32 x 256  GLA, fused     41.1 -> 41.5   53.0 -> 51.4
//     256 32 32 x 64   GLA            23.2 -> 22.4   28.3 -> 26.1
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sla.h"

namespace sla {

typedef __attribute__((ext_vector_type(4))) float d_f32x4;

namespace {

constexpr float kDecLog2e = 1.4426950408889634f;
constexpr int kDecThreads = 256;

struct DArgs {
    const void* q;
    const void* k;
    const void* v;
    const float* ql;
    const float* kl;
    const float* wq;        // fused gate projection: [H,dk] fp32 (then ql, kl are not read), else null
    const float* wk;        // [H,dk] fp32 or null (G^K = 1)
    const void* ld;
    const float* beta;
    float* state;
    void* out;
    int B, H, dv;
};

__device__ __forceinline__ float dec_exp(float x) { return __builtin_amdgcn_exp2f(x * kDecLog2e); }

template <bool BF16>
__device__ __forceinline__ float load_elem(const void* p, size_t i) {
    if constexpr (BF16)
        return __uint_as_float((uint32_t)((const uint16_t*)p)[i] << 16);
    else
        return ((const float*)p)[i];
}

// N adjacent elements starting at element i (N a multiple of 4; the address is 8- or 16-byte aligned), as wide loads
template <bool BF16, int N>
__device__ __forceinline__ void load_run(const void* p, size_t i, float (&x)[N]) {
    if constexpr (BF16) {
        typedef __attribute__((ext_vector_type(2))) uint32_t u2;
#pragma unroll
        for (int e = 0; e < N; e += 4) {
            const u2 t = *(const u2*)((const uint16_t*)p + i + e);
            x[e] = __uint_as_float(t.x << 16);
            x[e + 1] = __uint_as_float(t.x & 0xffff0000u);
            x[e + 2] = __uint_as_float(t.y << 16);
            x[e + 3] = __uint_as_float(t.y & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int e = 0; e < N; e += 4) {
            const d_f32x4 t = *(const d_f32x4*)((const float*)p + i + e);
            x[e] = t[0]; x[e + 1] = t[1]; x[e + 2] = t[2]; x[e + 3] = t[3];
        }
    }
}

__device__ __forceinline__ uint32_t dec_pack_bf16(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf2;
    bf2 t;
    t.x = (__bf16)lo;
    t.y = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, t);
}

// softmax over the H logits of one batch row, lane i holding logit i (lanes past H: -inf), evaluated for head h (Eq. 4);
// every lane of the wave returns it
__device__ __forceinline__ float decode_gate(float x, int H, int h, int lane) {
    float m = x;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    const float e = lane < H ? dec_exp(x - m) : 0.f;
    float s = e;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    return __shfl(e, h) / s;
}

// Sum over the row groups that share a wave (lanes NC4 apart hold the same columns), left in all of them.
template <int NC4>
__device__ __forceinline__ float wave_rows_sum(float x) {
#pragma unroll
    for (int o = NC4; o < 64; o <<= 1) x += __shfl_xor(x, o);
    return x;
}

// Which form of the gates an instantiation holds.  kLogits is the plain step alone, five workgroups of dk = 128 to a
// compute unit (B=32 H=16 128 x 128 GLA 10.3 / 17.2 -> 9.1 / 15.9 us, near / far; B=32 H=64 64 x 64 10.9 / 15.8 -> 9.3 / 15.2).
// kEither decides at run time, and the projection's registers leave three workgroups: the better where the state
// overflows the caches anyway, and the plain step's choice from 60 MB on (B=64 H=16 128 x 128 GLA 21.4 / 28.1 us,
// 22.1 / 27.7 by kLogits; 128 x 256 40.6 / 50.3 and 41.7 / 51.8).
enum Gates { kLogits, kProjected, kEither };

// One workgroup: `DS` adjacent value columns (slice blockIdx.x % slices) of one (batch, head).
template <bool BF16, int VAR, int DK, int DS, Gates GATES>
__global__ __launch_bounds__(kDecThreads) void sla_decode_kernel(const DArgs a) {
    constexpr int NC4 = DS / 4;             // threads along a row of the slice
    constexpr int NRG = kDecThreads / NC4;  // row groups
    constexpr int RPT = DK / NRG;           // rows per thread
    constexpr int NW = kDecThreads / 64;
    static_assert(NC4 <= 64 && DK % NRG == 0 && RPT >= 1, "rows divide among the row groups, a row lies in one wave");
    __shared__ float red[NW][DS];  // per-wave partial sums over the state rows

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // workgroups go round-robin over the eight XCDs: the slices of a head, which share its rows' memory pages and its
    // vectors, are placed on one of them
    const int slices = a.dv / DS, place = blockIdx.x >> 3, slice = place % slices;
    const int bh = (place / slices) * 8 + (blockIdx.x & 7), b = bh / a.H, h = bh % a.H;
    if (bh >= a.B * a.H) return;
    const int c4 = tid % NC4, rg = tid / NC4, row4 = a.dv / 4;

    const bool fused = GATES == kProjected || (GATES == kEither && a.wq);
    d_f32x4* srow = (d_f32x4*)(a.state + (size_t)bh * DK * a.dv + slice * DS) + c4;
    float qd[RPT], kd[RPT], ad[RPT], v4[4], ld_scalar = 0.f, bt = 0.f;
    d_f32x4 S[RPT];
    auto load_vectors = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const size_t d = (size_t)bh * DK + rg + NRG * i;
            qd[i] = load_elem<BF16>(a.q, d);
            kd[i] = load_elem<BF16>(a.k, d);
            if constexpr (VAR == SLA_GLA) ad[i] = load_elem<BF16>(a.ld, d);
        }
        load_run<BF16, 4>(a.v, (size_t)bh * a.dv + slice * DS + 4 * c4, v4);
        if constexpr (VAR == SLA_RETNET) ld_scalar = ((const float*)a.ld)[h];
        if constexpr (VAR == SLA_GDN) {
            ld_scalar = ((const float*)a.ld)[bh];
            bt = a.beta[bh];
        }
    };
    auto load_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) S[i] = srow[(size_t)(rg + NRG * i) * row4];
    };

    // Loads come back in the order they were issued, so what the gates are made of goes first: they are then formed
    // while the state tile and the token's vectors, all issued before anything waits, are still on their way.  kProjected
    // asks for the state first and for the vectors behind the projection, whose registers they then take: four workgroups
    // to a compute unit instead of three.  It is chosen where the state fits the caches (GLA, near: B=32 H=64 64 x 64
    // 16.8 -> 15.4 us, B=100 H=8 128 x 64 10.1 -> 8.3; delta rule, far: B=24 H=16 128 x 256 24.5 -> 22.7), and for GLA
    // where the projection takes more than the one round of loads that goes out ahead of the state, beyond 16 heads
    // (B=16 H=64 128 x 256 53.4 -> 48.1, B=256 H=4 128 x 128 22.6 -> 22.0 near, 28.9 -> 29.7 far).
    constexpr int TPH = DK >= 64 ? 16 : 8, EPT = DK / TPH;  // fused projection: threads per head, elements per thread
    const int sub = tid % TPH;
    int h2 = tid / TPH;
    float xq[EPT], xk[EPT], wq[EPT], wk[EPT], lq = -INFINITY, lk = -INFINITY;
    auto load_projection = [&]() __attribute__((always_inline)) {
        const size_t at = ((size_t)b * a.H + h2) * DK + sub * EPT, wat = (size_t)h2 * DK + sub * EPT;
        load_run<BF16, EPT>(a.q, at, xq);
        load_run<false, EPT>(a.wq, wat, wq);
        if (a.wk) {
            load_run<BF16, EPT>(a.k, at, xk);
            load_run<false, EPT>(a.wk, wat, wk);
        }
    };
    if constexpr (GATES == kProjected) load_state();
    if (fused) {
        if (h2 < a.H) load_projection();
    } else if (lane < a.H) {
        lq = a.ql[(size_t)b * a.H + lane];
        if (a.kl) lk = a.kl[(size_t)b * a.H + lane];
    }
    if constexpr (GATES != kProjected) {
        load_vectors();
        load_state();
    }

    if (fused) {
        // Fused gate projection (Eq. 4 needs the logits of every head of the token): TPH threads per head (16; 8 for
        // dk = 32), each thread DK/TPH >= 4 adjacent elements of q[b,h',:] . W_GQ[:,h'] and k[b,h',:] . W_GK[:,h'],
        // summed over the TPH threads with shuffles -- 2 H dk multiply-adds against the dk dv of the state update, and
        // one launch less in front of every decode step.
        __shared__ float lg[2][64];
        while (h2 < a.H) {
            float sq = 0.f, sk = 0.f;
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                sq += xq[e] * wq[e];
                if (a.wk) sk += xk[e] * wk[e];
            }
#pragma unroll
            for (int o = TPH / 2; o >= 1; o >>= 1) {
                sq += __shfl_xor(sq, o);
                sk += __shfl_xor(sk, o);
            }
            if (sub == 0) {
                lg[0][h2] = sq;
                lg[1][h2] = sk;
            }
            h2 += kDecThreads / TPH;
            if (h2 < a.H) load_projection();
        }
        __syncthreads();
        if (lane < a.H) {
            lq = lg[0][lane];
            lk = lg[1][lane];
        }
    }
    if constexpr (GATES == kProjected) load_vectors();
    const float gq = decode_gate(lq, a.H, h, lane);
    const float gk = (fused ? (const void*)a.wk : (const void*)a.kl) ? decode_gate(lk, a.H, h, lane) : 1.f;

    const float a_scalar = dec_exp(ld_scalar);
    // Sec. 5.1: the write.  RetNet / GLA: S <- a S + (G^K k)^T v.  Delta rule: Sb = a S, u = beta (G^K v - k Sb),
    // S <- Sb + k^T u, which needs k Sb over all rows first.
    float w4[4];  // what is added as k_d * w
    if constexpr (VAR == SLA_GDN) {
        float ks[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                S[i][j] *= a_scalar;
                ks[j] += kd[i] * S[i][j];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) ks[j] = wave_rows_sum<NC4>(ks[j]);
        if (lane < NC4) *(d_f32x4*)&red[wave][4 * c4] = d_f32x4{ks[0], ks[1], ks[2], ks[3]};
        __syncthreads();
        d_f32x4 t = *(const d_f32x4*)&red[0][4 * c4];
#pragma unroll
        for (int g = 1; g < NW; ++g) t += *(const d_f32x4*)&red[g][4 * c4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w4[j] = bt * (gk * v4[j] - t[j]);
        __syncthreads();
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) w4[j] = gk * v4[j];
    }

    float y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const float al = VAR == SLA_GLA ? dec_exp(ad[i]) : a_scalar;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float decayed = VAR == SLA_GDN ? S[i][j] : al * S[i][j];
            S[i][j] = decayed + kd[i] * w4[j];
            y[j] += qd[i] * S[i][j];  // Eq. 6: the read-out uses the updated state
        }
        srow[(size_t)(rg + NRG * i) * row4] = S[i];
    }

    // out = G^Q (q S): sum the row groups
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = wave_rows_sum<NC4>(y[j]);
    if (lane < NC4) *(d_f32x4*)&red[wave][4 * c4] = d_f32x4{y[0], y[1], y[2], y[3]};
    __syncthreads();
    if (tid < DS / 2) {
        float o0 = 0.f, o1 = 0.f;
#pragma unroll
        for (int g = 0; g < NW; ++g) {
            o0 += red[g][2 * tid];
            o1 += red[g][2 * tid + 1];
        }
        o0 *= gq;
        o1 *= gq;
        const size_t at = ((size_t)bh * a.dv + slice * DS) / 2 + tid;
        if constexpr (BF16)
            ((uint32_t*)a.out)[at] = dec_pack_bf16(o0, o1);
        else
            ((float2*)a.out)[at] = make_float2(o0, o1);
    }
}

// The whole state below 60 MB, well inside the caches' capacity: see Gates.
template <int DK>
bool small_state(const DArgs& a) {
    return (size_t)a.B * a.H * DK * a.dv * 4 < (size_t)60 << 20;
}

// Value columns per workgroup (the figures are in the file header).
template <int VAR, int DK>
int slice_width(const DArgs& a, bool overlap) {
    const size_t heads = (size_t)a.B * a.H, narrow = heads * (a.dv / 64);  // workgroups at 64 columns
    int ds = 64;
    if (narrow <= (a.wq ? 1 : 2) * (size_t)DK) {
        ds = 32;
    } else if (a.wq && narrow > 256) {  // every slice repeats the projection: eight state rows per thread, or sixteen
        ds = 8192 / DK;
        if (narrow > 512 && ds < 128 && (small_state<DK>(a) || (VAR == SLA_GLA && a.H > 32))) ds = 128;
    }
    if (ds > a.dv) ds = a.dv;
    // One workgroup per head reads all of the head's inputs before it writes any of its out, so that out may lie on them;
    // and a launch holds fewer than 2^32 threads.
    if (overlap || (heads + 7) / 8 * 8 * (a.dv / ds) * kDecThreads > 0xffffffffu) ds = a.dv;
    return ds;
}

template <bool BF16, int VAR, int DK, int DS>
void launch_width(const DArgs& a, hipStream_t stream) {
    const dim3 grid((unsigned)(((size_t)a.B * a.H + 7) / 8 * 8 * (a.dv / DS))), block(kDecThreads);
    const bool small = small_state<DK>(a);
    if (a.wq && (small || (VAR == SLA_GLA && a.H > 16))) {
        hipLaunchKernelGGL((sla_decode_kernel<BF16, VAR, DK, DS, kProjected>), grid, block, 0, stream, a);
        return;
    }
    if constexpr (DS <= 64) {
        if (!a.wq && small) {
            hipLaunchKernelGGL((sla_decode_kernel<BF16, VAR, DK, DS, kLogits>), grid, block, 0, stream, a);
            return;
        }
    }
    hipLaunchKernelGGL((sla_decode_kernel<BF16, VAR, DK, DS, kEither>), grid, block, 0, stream, a);
}

template <bool BF16, int VAR, int DK>
int launch_dv(const DArgs& a, hipStream_t stream) {
    const size_t es = BF16 ? 2 : 4, heads = (size_t)a.B * a.H;
    auto on_out = [&](const void* x, size_t bytes) {
        const uintptr_t o = (uintptr_t)a.out, i = (uintptr_t)x;
        return x && o < i + bytes && i < o + heads * a.dv * es;
    };
    const bool overlap = on_out(a.q, heads * DK * es) || on_out(a.k, heads * DK * es) || on_out(a.v, heads * a.dv * es) ||
                         (VAR == SLA_GLA && on_out(a.ld, heads * DK * es)) ||
                         (VAR == SLA_GDN && (on_out(a.ld, heads * 4) || on_out(a.beta, heads * 4)));
    switch (slice_width<VAR, DK>(a, overlap)) {
        case 32: launch_width<BF16, VAR, DK, 32>(a, stream); break;
        case 64: launch_width<BF16, VAR, DK, 64>(a, stream); break;
        case 128: launch_width<BF16, VAR, DK, 128>(a, stream); break;
        case 256: launch_width<BF16, VAR, DK, 256>(a, stream); break;
        default: return SLA_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? SLA_OK : SLA_ERR_HIP;
}

template <bool BF16, int VAR>
int launch_dk(const DArgs& a, int dk, hipStream_t stream) {
    switch (dk) {
        case 32: return launch_dv<BF16, VAR, 32>(a, stream);
        case 64: return launch_dv<BF16, VAR, 64>(a, stream);
        case 128: return launch_dv<BF16, VAR, 128>(a, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}

template <bool BF16>
int launch_var(const DArgs& a, int variant, int dk, hipStream_t stream) {
    switch (variant) {
        case SLA_RETNET: return launch_dk<BF16, SLA_RETNET>(a, dk, stream);
        case SLA_GLA: return launch_dk<BF16, SLA_GLA>(a, dk, stream);
        case SLA_GDN: return launch_dk<BF16, SLA_GDN>(a, dk, stream);
        default: return SLA_ERR_UNSUPPORTED;
    }
}

}  // namespace

int launch_decode(const sla_params& p, const void* q, const void* k, const void* v, const float* ql, const float* kl,
                  const float* wq, const float* wk, const void* ld, const float* beta, float* state, void* out,
                  hipStream_t stream) {
    DArgs a;
    a.q = q; a.k = k; a.v = v; a.ql = ql; a.kl = kl; a.wq = wq; a.wk = wk; a.ld = ld; a.beta = beta; a.state = state;
    a.out = out;
    a.B = p.B; a.H = p.H; a.dv = p.dv;
    if (p.dtype == SLA_BF16) return launch_var<true>(a, p.variant, p.dk, stream);
    return launch_var<false>(a, p.variant, p.dk, stream);
}

}  // namespace sla
