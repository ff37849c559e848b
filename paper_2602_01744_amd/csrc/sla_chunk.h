// Chunk-parallel schedule of RetNet / GLA on bf16 tensors: what its kernels share.  The tokens of a sequence are cut into
// chunks of 64.  sla_chunk_state.hip carries the states over the chunks and leaves, for every chunk, the state entering
// it (S) and the gradient with respect to the state behind it (X), in bf16 operand pieces; everything else of a chunk
// depends on these and on its own rows, so one workgroup per chunk and head makes all outputs of the chunk.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "sla.h"
#include "sla_chunk_plan.h"
#include "sla_lane_ops.h"

namespace sla {
namespace chk {

using namespace lane_ops;

constexpr int kChunk = kChunkTokens;  // tokens per chunk: four 16-token blocks, the unit within which GLA's decay products are formed

struct Args {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const uint16_t* dout;
    const uint16_t* ld;      // GLA: [B,T,H,dk]
    const float* ld_head;    // RetNet: [H]
    const float* gq;         // gates [B,T,H]
    const float* gk;
    const float* s0;         // [B,H,dk,dv] or null
    const float* dsf;        // cotangent of the final state or null
    float* ds0;              // gradient of the initial state or null
    float* end;              // GLA with dsf: [B,H][dv/32][dk] rowsum(dsf * S) over 32 value columns each, S entering the last chunk
    u4* S;                   // operand pieces of the state entering a chunk, see piece()
    u4* X;                   // ... of the gradient with respect to the state behind it
    uint16_t* dq;
    uint16_t* dk;
    uint16_t* dv;
    uint16_t* dld;
    float* dgq;              // [B,T,H] gradients of the gates
    float* dgk;
    int B, T, H;             // T: tokens per batch row, or of the whole packed batch
    const int* cu;           // packed batch: sequence b is tokens cu[b] .. cu[b+1]-1 of T; else null
    bool head_major;         // wide tensors are [B,H,T,d]
    // The part of the batch this launch works on: sequences b0 .. b0+nb-1, heads h0 .. h0+nh-1.  slots: chunks of the
    // part per head; the states of slot s, head h0 + i lie at (s * nh + i).
    int b0, nb, h0, nh, slots, nchunk;
};

struct Sequence {
    int T;         // tokens
    size_t tok0;   // first token, counted over the batch
    int slot0;     // slot of its first chunk
};
__device__ __forceinline__ Sequence sequence(const Args& a, int b) {
    if (a.cu) {  // offsets are clamped into the tensors whatever cu holds
        const int start = min(max(a.cu[b], 0), a.T), end = min(max(a.cu[b + 1], start), a.T);
        return Sequence{end - start, (size_t)start, start / kChunk + b};
    }
    return Sequence{a.T, (size_t)b * a.T, (b - a.b0) * a.nchunk};
}

// The sequence and chunk of a slot; false: it has none.  Packed sequences' first slots grow with their number, so a wave
// narrows them down 64 at a time: one step for 64 sequences, two for 4096.  (A workgroup looking at all of them: 16384 tokens
// in as many sequences, RetNet H=8 64 x 64, 5140 us a backward call against 2127; in 1024, H=16 128 x 128, 951 against 922.)
__device__ __forceinline__ bool chunk_of(const Args& a, int slot, int& b, int& chunk) {
    if (!a.cu) {
        b = a.b0 + slot / a.nchunk;
        chunk = slot % a.nchunk;
        return true;
    }
    int lo = 0, n = a.B;
    while (true) {
        const int step = (n + 63) / 64, i = (int)(threadIdx.x & 63) * step;
        const bool before = i < n && min(max(a.cu[lo + min(i, n - 1)], 0), a.T) / kChunk + lo + i <= slot;
        const int count = __builtin_popcountll(__ballot(before));
        if (count == 0) return false;
        lo += (count - 1) * step;
        if (step == 1) break;
        n = min(step, n - (count - 1) * step);
    }
    b = __builtin_amdgcn_readfirstlane(lo);
    const Sequence s = sequence(a, b);
    chunk = slot - s.slot0;
    return chunk >= 0 && chunk < (s.T + kChunk - 1) / kChunk;
}

__device__ __forceinline__ float bf_at(const u4& x, int i) { return (i & 1) ? bf_hi(x[i >> 1]) : bf_lo(x[i >> 1]); }
__device__ __forceinline__ u4 pack8(f4 x, f4 y) {
    return u4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(y[0], y[1]), pack2(y[2], y[3])};
}
__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ s8 op(u4 x) { return __builtin_bit_cast(s8, x); }
// inclusive sums over the 16 lanes of a row (tokens), from lane 15 down
__device__ __forceinline__ float row_suffix(float x) {
    x += dpp<0x101>(x);
    x += dpp<0x102>(x);
    x += dpp<0x104>(x);
    x += dpp<0x108>(x);
    return x;
}
__device__ __forceinline__ float row_last(float x) { return dpp<0x15F>(x); }   // lane 15 of the row, to all
__device__ __forceinline__ float row_first(float x) { return dpp<0x150>(x); }  // lane 0 of the row, to all

// Rows of one sequence and head through a buffer descriptor that ends with the sequence: tokens past it read as zero.
constexpr uint32_t kRsrcWord3 = 0x00020000u;  // raw buffer, 32-bit data format
struct Rows {
    __amdgpu_buffer_rsrc_t d;
    int off, step;  // bytes: column 0 of token 0, and from token to token
    __device__ __forceinline__ u4 load(int t, int col) const {
        return __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(d, off + t * step + 2 * col, 0, 0));
    }
    __device__ __forceinline__ void put(int t, int col, u4 x) const {  // tokens past the end are dropped
        __builtin_amdgcn_raw_buffer_store_b128(x, d, off + t * step + 2 * col, 0, 0);
    }
};
template <int D>
__device__ __forceinline__ Rows rows_of(const Args& a, const uint16_t* x, const Sequence& s, int b, int h) {
    const size_t base = a.head_major ? ((size_t)b * a.H + h) * a.T * D : s.tok0 * a.H * D;
    const int step = (a.head_major ? 1 : a.H) * D * 2;
    return Rows{__builtin_amdgcn_make_buffer_rsrc((void*)(x + base), 0, s.T * step, kRsrcWord3), a.head_major ? 0 : h * D * 2, step};
}
__device__ __forceinline__ Rows scalars_of(const Args& a, const float* x, const Sequence& s, int h) {
    return Rows{__builtin_amdgcn_make_buffer_rsrc((void*)(x + s.tok0 * a.H), 0, s.T * a.H * 4, kRsrcWord3), h * 4, a.H * 4};
}
__device__ __forceinline__ float load_scalar(const Rows& x, int t) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(x.d, x.off + t * x.step, 0, 0));
}

// A state in operand pieces: piece (tile, c), tile = 16 key dimensions, c = 32 value columns, is one 16-byte unit per lane,
// 1 KiB without gaps per load or store.  Lane (r, g) of tile 2w + i holds key dimension 32w + 8 (r / 4) + 4i + r % 4, value
// columns 32c + 8g .. + 7.  (With that order of a tile pair's rows a lane's two accumulators are eight adjacent
// dimensions of one token: 16-byte loads and stores of the rows, and the scans over tokens run along lanes.)
template <int DK, int DV>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pieces_of(u4* states, size_t state) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(states + state * (DK * DV / 8)), 0, DK * DV * 2, kRsrcWord3);
}
template <int DV>
__device__ __forceinline__ int piece(int tile, int c) { return (tile * (DV / 32) + c) * 1024; }  // bytes
__device__ __forceinline__ int key_of(int i, int r) { return 8 * (r >> 2) + 4 * i + (r & 3); }

// the lower triangle's ten 16 x 16 tiles (t block, j block), dealt to the waves in turn
constexpr uint64_t kTileT = 0x3323213210ull, kTileJ = 0x0102103210ull;
static_assert(((kTileT >> 36) & 15) == 3 && ((kTileJ >> 36) & 15) == 0, "ten tiles");

// 16-byte unit u of row `row` of an LDS array with U units per row: rows that a group of 16 lanes reads together lie on
// different banks.
template <int U>
__device__ __forceinline__ int unit_at(int row, int u) {
    if constexpr (U == 16) return row * U + (u ^ (row & 15));
    if constexpr (U == 8) return row * U + (u ^ ((row >> 1) & 7));
    return row * U + (u ^ ((row >> 2) & 3));
}

// Lets KERNEL use that much dynamic LDS: once per device and kernel (bit d = done on device d); not a stream operation.
template <auto KERNEL>
static bool allow_lds(int bytes) {
    static std::atomic<uint64_t> configured{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return false;
    }
    if (!((configured.load(std::memory_order_acquire) >> dev) & 1u)) {
        if (hipFuncSetAttribute((const void*)KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        configured.fetch_or(uint64_t(1) << dev, std::memory_order_release);
    }
    return true;
}

}  // namespace chk
}  // namespace sla
