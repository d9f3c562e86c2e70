// fp32 grouped SwiGLU FFN over the united experts (each expert an FFN of
// Sec. 2.1; SwiGLU form): the layer's reference-precision path. Products and
// sums are fp32 throughout (fp32 MFMA: fused multiply-adds into fp32).
//
// A call of this path is small (tens to hundreds of rows), so it is bound by
// the latency of its dependent loads and by how many CUs take part, not by
// MFMA or bandwidth. One workgroup therefore owns a small tile, 32 rows x 32
// output columns (of both matrices for gate/up), and its eight waves split K:
// every wave loads its share of the tile's rows straight into registers, a
// batch at a time with the next one in flight, and the eight partial tiles
// meet in LDS, where they are added in wave order (deterministic).
// The tiny layer (T = 64, top-2, d = 256, d_ff = 512, 4 united
// experts), by the kernel trace: gate/up 126 -> 14 us, down 75 -> 8.8 us against one output
// element per thread (a serial chain of uncoalesced loads).
//
// k-order: lane half h = lane / 32 of a 32x32x2 MFMA supplies one k value; a
// lane loads 16 bytes, so MFMA e of unit u multiplies columns 8u + e (half 0)
// and 8u + 4 + e (half 1), the same for both operands. d and d_ff are
// multiples of 8, so there is no partial unit.
#include "bmoe_common.h"

namespace bmoe {
namespace {

constexpr int kFThreads = 512;
constexpr int kFWaves = kFThreads / 64;
constexpr int kFTile = 32;    // rows, and output columns, of a workgroup
constexpr int kFUnit = 8;     // K columns of a unit (one 16-byte load per lane)
constexpr int kFBatch = 4;    // units in flight per operand and step
constexpr int kFPad = 34;     // floats per row of a partial tile in LDS (even: read two at a time)
constexpr int kFMaxY = 32768;  // most row tiles of a grid; workgroups then take several

struct F32Params {
    const float* A;   // [rows_cap or a_count, K]
    const float* B0;  // [n_seg, N, K]
    const float* B1;  // [n_seg, N, K] (gated: W_up)
    float* C;         // [rows_cap, N]
    const int32_t* offsets;
    int n_seg, rows_cap, N, K;
    const int32_t* a_rows;  // gathered A: row r is A[a_rows[r]] (A has a_count rows); nullptr: row r is A[r]
    int a_count;
};

// The segment and rows [m0, m_end) of row tile m (32 rows, segments in
// order); false past the last tile. Every wave computes it for itself.
__device__ __forceinline__ bool f32_tile(const F32Params& p, int m, int lane, int& seg, int& m0, int& m_end) {
    int base = 0;
    for (int s0 = 0; s0 < p.n_seg; s0 += kWave) {
        const int s = s0 + lane;
        int beg = 0, end = 0;
        if (s < p.n_seg) {
            beg = min(max(p.offsets[s], 0), p.rows_cap);
            end = min(max(p.offsets[s + 1], beg), p.rows_cap);
        }
        const int cnt = ceil_div(end - beg, kFTile);
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        const unsigned long long past = __ballot(base + incl > m);
        if (past != 0ull) {
            const int src = __ffsll(past) - 1;
            seg = __builtin_amdgcn_readfirstlane(s0 + src);
            m0 = __builtin_amdgcn_readfirstlane(__shfl(beg + (m - (base + incl - cnt)) * kFTile, src));
            m_end = __builtin_amdgcn_readfirstlane(__shfl(end, src));
            return true;
        }
        base += __shfl(incl, kWave - 1);
    }
    return false;
}

template <int NMAT>
struct F32Batch {
    float4 a[kFBatch];
    float4 b[NMAT][kFBatch];
};

// units u0 .. u0 + kFBatch - 1 of this lane's rows, as many as lie below u1
// (the loads of the others repeat unit u1 - 1 and are not used: a branch
// around a load would cost its latency)
template <int NMAT>
__device__ __forceinline__ void f32_load(F32Batch<NMAT>& v, const float* ar, const float* const (&br)[NMAT], int u0,
                                         int u1) {
#pragma unroll
    for (int j = 0; j < kFBatch; ++j) {
        const size_t o = (size_t)min(u0 + j, u1 - 1) * kFUnit;
        v.a[j] = *(const float4*)(ar + o);
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat) v.b[mat][j] = *(const float4*)(br[mat] + o);
    }
}

template <int NMAT>
__device__ __forceinline__ void f32_mfma(f32x16 (&acc)[NMAT], const F32Batch<NMAT>& v, int u0, int u1) {
#pragma unroll
    for (int j = 0; j < kFBatch; ++j) {
        if (u0 + j >= u1) break;  // (the same for the whole wave)
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat)
            acc[mat] = __builtin_amdgcn_mfma_f32_32x32x2f32(v.a[j].x, v.b[mat][j].x, acc[mat], 0, 0, 0);
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat)
            acc[mat] = __builtin_amdgcn_mfma_f32_32x32x2f32(v.a[j].y, v.b[mat][j].y, acc[mat], 0, 0, 0);
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat)
            acc[mat] = __builtin_amdgcn_mfma_f32_32x32x2f32(v.a[j].z, v.b[mat][j].z, acc[mat], 0, 0, 0);
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat)
            acc[mat] = __builtin_amdgcn_mfma_f32_32x32x2f32(v.a[j].w, v.b[mat][j].w, acc[mat], 0, 0, 0);
    }
}

template <bool GATED>
__global__ __launch_bounds__(kFThreads) void ffn_f32_kernel(F32Params p) {
    constexpr int NMAT = GATED ? 2 : 1;
    __shared__ __align__(16) float part[kFWaves][NMAT][kFTile * kFPad];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int N = p.N, K = p.K;
    const int l32 = lane & 31, half = lane >> 5;
    const int n0 = (int)blockIdx.x * kFTile;
    // (a kernel this short pays for its own instruction fetches: no division, one copy of the loop)
    for (int t = blockIdx.y;; t += gridDim.y) {
        int seg, m0, m_end;
        if (!f32_tile(p, t, lane, seg, m0, m_end)) return;
        // this wave's units of K
        const int nu = K / kFUnit;
        const int u0 = nu * wave / kFWaves, u1 = nu * (wave + 1) / kFWaves;
        const float* ar = p.A + (size_t)gathered_row(p.a_rows, p.a_count, min(m0 + l32, m_end - 1)) * K + half * 4;
        const size_t brow = ((size_t)seg * N + min(n0 + l32, N - 1)) * K + half * 4;
        const float* br[NMAT];
        br[0] = p.B0 + brow;
        if constexpr (GATED) br[NMAT - 1] = p.B1 + brow;
        f32x16 acc[NMAT];
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mat][i] = 0.f;
        if (u0 < u1) {  // (K of fewer than eight units leaves waves without one)
            F32Batch<NMAT> v0, v1;
            f32_load<NMAT>(v0, ar, br, u0, u1);
            for (int u = u0; u < u1; u += 2 * kFBatch) {
                f32_load<NMAT>(v1, ar, br, u + kFBatch, u1);
                f32_mfma<NMAT>(acc, v0, u, u1);
                f32_load<NMAT>(v0, ar, br, u + 2 * kFBatch, u1);
                f32_mfma<NMAT>(acc, v1, u + kFBatch, u1);
            }
        }
#pragma unroll
        for (int mat = 0; mat < NMAT; ++mat)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                part[wave][mat][(8 * (i >> 2) + 4 * half + (i & 3)) * kFPad + l32] = acc[mat][i];
        __syncthreads();
        // each thread sums two neighbouring columns of one row, in wave order
        const int r = tid / (kFTile / 2), c = (tid % (kFTile / 2)) * 2;
        const int gm = m0 + r, gn = n0 + c;
        if (gm < m_end && gn < N) {
            float2 v[NMAT];
#pragma unroll
            for (int mat = 0; mat < NMAT; ++mat) {
                v[mat] = *(const float2*)&part[0][mat][r * kFPad + c];
#pragma unroll
                for (int w = 1; w < kFWaves; ++w) {
                    const float2 o = *(const float2*)&part[w][mat][r * kFPad + c];
                    v[mat].x += o.x;
                    v[mat].y += o.y;
                }
            }
            if constexpr (GATED) {
                v[0].x = v[0].x / (1.f + expf(-v[0].x)) * v[NMAT - 1].x;
                v[0].y = v[0].y / (1.f + expf(-v[0].y)) * v[NMAT - 1].y;
            }
            *(float2*)(p.C + (size_t)gm * N + gn) = v[0];  // (N is even: no half pair)
        }
        __syncthreads();  // the next tile rewrites the partial tiles
    }
}

template <bool GATED>
hipError_t launch_f32(const F32Params& p, hipStream_t s) {
    // the most row tiles that offsets over rows_cap rows can name
    const int64_t mt = ceil_div64(p.rows_cap, kFTile) + (p.n_seg < p.rows_cap ? p.n_seg : p.rows_cap);
    const dim3 grid((unsigned)ceil_div(p.N, kFTile), (unsigned)(mt < kFMaxY ? mt : kFMaxY));
    hipLaunchKernelGGL((ffn_f32_kernel<GATED>), grid, dim3(kFThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_f32(const FfnArgs& a, hipStream_t s, int part) {
    if (part != 2) {
        F32Params g{(const float*)a.a, (const float*)a.w_gate, (const float*)a.w_up, (float*)a.h, a.offsets,
                    a.n_seg, a.rows_cap, a.d_ff, a.d, a.a_rows, a.a_count};
        hipError_t e = launch_f32<true>(g, s);
        if (e != hipSuccess) return e;
    }
    if (part != 1) {
        F32Params g{(const float*)a.h, (const float*)a.w_down, nullptr, (float*)a.y, a.offsets,
                    a.n_seg, a.rows_cap, a.d, a.d_ff, nullptr, 0};
        return launch_f32<false>(g, s);
    }
    return hipSuccess;
}

}  // namespace bmoe
