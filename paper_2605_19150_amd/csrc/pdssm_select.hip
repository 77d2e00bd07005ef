// pdssm_select.hip -- the selection front end of the scan (Sec. 3.1 eqs. (5)-(8),
// App. E.2.1):
//
//   maps      pi[h,k,j] = argmax_i M[h,k,i,j]   (column argmax of the dense
//                                                dictionary, once per step of
//                                                the optimizer)
//   routing   logits[t,h,k] = sum_d u[t,d] S[h,k,d],   idx[t,h] = argmax_k logits[t,h,k]
//
// Ties go to the first maximal index (numpy's and torch's rule).
//
// k_route: the routing product on the matrix cores (v_mfma_f32_32x32x16_bf16:
// bf16 operands, fp32 accumulation) with the argmax fused into the epilogue.
// A workgroup computes a 128-token x (whole heads, at most 256 columns)
// tile: four waves own 64 x 128 blocks (2 x 4 tiles of 32 x 32).  The
// contraction goes in slices of 64, copied by the workgroup into LDS (two
// stages: the next slice's global loads run while the current one is
// multiplied).  The fp32 tile then goes to LDS in two halves, from where it is
// written out coalesced and each (token, head) takes its argmax, so the
// logits are read back from nowhere.
#include "pdssm_device.h"
#include "pdssm_project_rule.h"
#include "pdssm_select.h"

#include <type_traits>

namespace pdssm {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kRouteTM = 128;  // tokens per workgroup
constexpr int kRouteTN = 256;  // column capacity per workgroup (whole heads)
constexpr int kRouteKS = 64;   // contraction slice staged in LDS (one 128-byte line per row)
constexpr int kRoutePitch = kRouteKS + 8;  // padded LDS row (bf16): 16-byte reads without bank conflicts
constexpr int kRouteStageElems = (kRouteTM + kRouteTN) * kRoutePitch;
// two stages of bf16; the epilogue tile (half the tokens, fp32) aliases them
constexpr size_t kRouteStages = 2 * kRouteStageElems * 2, kRouteTile = (size_t)kRouteTM / 2 * kRouteTN * 4;
constexpr size_t kRouteLds = kRouteStages > kRouteTile ? kRouteStages : kRouteTile;

// Lane layout of v_mfma_f32_32x32x16_bf16: lane l supplies A[l%32][8(l/32) .. 8(l/32)+7]
// and B[8(l/32) .. +7][l%32]; accumulator element r of lane l is
// C[8(r/4) + 4(l/32) + r%4][l%32].
// Waves form a 2 x 2 grid of 64-token x 128-column blocks.  Each slice of 64
// of the contraction is copied by the whole workgroup from global memory
// (coalesced 16-byte chunks, rows past the tensor clamped, chunks past the
// contraction zero) into one of two LDS stages while the other stage is
// multiplied; one barrier per slice.
__global__ __launch_bounds__(256) void k_route(RouteArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    uint16_t* stage_base = reinterpret_cast<uint16_t*>(lds);
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wm = wv >> 1, wn = wv & 1;
    const int hpb = kRouteTN / a.K;              // heads per workgroup
    const int h0 = blockIdx.y * hpb;
    const int nh = min(hpb, a.H - h0);
    const int ncol = nh * a.K;                   // valid columns of this tile
    const int m0 = blockIdx.x * kRouteTM;
    const int HK = a.H * a.K;

    f32x16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // copy plan: the stage holds kRouteTM rows of u then kRouteTN rows of S,
    // kRouteKS/8 chunks of 16 bytes per row; thread t takes chunks t, t + 256, ...
    constexpr int kCpr = kRouteKS / 8;
    constexpr int kChunks = (kRouteTM + kRouteTN) * kCpr;
    constexpr int kPer = kChunks / 256;
    static_assert(kChunks % 256 == 0, "whole chunks per thread");
    const uint16_t* src[kPer];
    int dst[kPer], col[kPer];
#pragma unroll
    for (int c = 0; c < kPer; ++c) {
        const int e = threadIdx.x + 256 * c;
        const int row = e / kCpr, ch = e % kCpr;
        col[c] = 8 * ch;
        dst[c] = row * kRoutePitch + 8 * ch;
        if (row < kRouteTM) {
            src[c] = a.u + (size_t)min(m0 + row, a.T - 1) * a.Dm;
        } else {
            const int n = min(row - kRouteTM, ncol - 1);
            src[c] = a.S + ((size_t)h0 * a.K + n) * a.Dm;
        }
    }
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    u32x4 reg[kPer];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int c = 0; c < kPer; ++c) {
            const int k = k0 + col[c];
            reg[c] = k < a.Dm ? *reinterpret_cast<const u32x4*>(src[c] + k) : u32x4{0, 0, 0, 0};
        }
    };
    auto store = [&](int st) {
        uint16_t* base = stage_base + st * kRouteStageElems;
#pragma unroll
        for (int c = 0; c < kPer; ++c) *reinterpret_cast<u32x4*>(base + dst[c]) = reg[c];
    };

    const int nslice = (a.Dm + kRouteKS - 1) / kRouteKS;
    const int c0 = wn * 128;  // this wave's first column of the tile
    const bool work = c0 < ncol;
    fetch(0);
    store(0);
    __syncthreads();
    const int kl = 8 * (lane >> 5);
    for (int sl = 0; sl < nslice; ++sl) {
        if (sl + 1 < nslice) fetch((sl + 1) * kRouteKS);
        if (work) {
            const uint16_t* As = stage_base + (sl & 1) * kRouteStageElems;
            const uint16_t* Bs = As + kRouteTM * kRoutePitch;
#pragma unroll
            for (int ks = 0; ks < kRouteKS; ks += 16) {
                bf16x8 A[2], B[4];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    A[i] = *reinterpret_cast<const bf16x8*>(As + (wm * 64 + 32 * i + (lane & 31)) * kRoutePitch + ks + kl);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    B[j] = *reinterpret_cast<const bf16x8*>(Bs + (c0 + 32 * j + (lane & 31)) * kRoutePitch + ks + kl);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[i], B[j], acc[i][j], 0, 0, 0);
            }
        }
        if (sl + 1 < nslice) store((sl + 1) & 1);
        __syncthreads();
    }

    float(*tile)[kRouteTN] = reinterpret_cast<float(*)[kRouteTN]>(lds);  // aliases the stages
    for (int half = 0; half < 2; ++half) {
        if (half) __syncthreads();  // the first half's readers are done
        if (wm == half && work) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        tile[32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)][c0 + 32 * j + (lane & 31)] =
                            acc[i][j][r];
        }
        __syncthreads();
        const int mb = m0 + half * (kRouteTM / 2);
        const int nm = max(0, min(kRouteTM / 2, a.T - mb));
        // logits: row m of the tile is ncol contiguous floats of the output
        if (a.logits)
            for (int e = threadIdx.x; e < nm * ncol; e += 256) {
                const int m = e / ncol, c = e - m * ncol;
                a.logits[(size_t)(mb + m) * HK + (size_t)h0 * a.K + c] = tile[m][c];
            }
        // argmax per (token, head): first maximal index
        for (int e = threadIdx.x; e < nm * nh; e += 256) {
            const int m = e / nh, hh = e - m * nh;
            const float* v = &tile[m][hh * a.K];
            int best = 0;
            float bv = v[0];
            for (int k = 1; k < a.K; ++k)
                if (v[k] > bv) bv = v[k], best = k;
            a.idx[(size_t)(mb + m) * a.H + h0 + hh] = best;
        }
    }
}

// ------------------------------------------------------------------ k_project_dma
// The routing product -- and the token projections b, c and the diagonal
// generator, as further column tiles of the same product -- for contraction
// sizes that are a multiple of 32, with
// direct buffer-to-LDS loads (buffer_load_dwordx4 ... lds: every lane of a
// wave moves 16 bytes to LDS at a wave-uniform base + 16 * lane), so that
// several slices are in flight without holding them in registers.  Rows past
// the end of u or S lie past their buffer descriptors and read as 0.
//
// A workgroup computes BM tokens x 256 columns (whole heads) with eight
// waves in a WGM x WGN grid.  The contraction goes in slices of 32 through
// NS = 4 LDS stages: while slice s is multiplied, slices s+1 .. s+3 are
// loading.  A stage holds BM rows of u, then 256 rows of S, 64 bytes of each;
// every 16 consecutive rows form a 1 KB block laid out chunk-major (byte
// (r/16)*1024 + c*256 + (r%16)*16 for row r, 16-byte chunk c), which is
// exactly what one wave-wide load instruction writes (lane l: row l%16, chunk
// l/16) and makes the operand reads (32 rows at one chunk) conflict-free.
// (Measured: loads of half cache lines, as here, reach about half the L2 rate
// of full ones, and the slices' loads set the pace of the kernel.)
//
// Tiles are numbered so that each XCD (workgroups are dealt round-robin over
// the 8 XCDs) takes a contiguous range, all column tiles of a few token tiles
// at a time: u streams from HBM once and the rows of S are shared in L2.
typedef __attribute__((address_space(3))) void* lds_void_t;

// One wave-wide 16-byte-per-lane load from a buffer into LDS at dst + 16*lane.
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, unsigned char* dst, uint32_t voff,
                                           uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t)dst, 16, voff, soff, 0, 0);
}

template <int BM>
struct RouteDma {
    static constexpr int BN = 256, BK = 32, NS = 4, NW = 8;
    static constexpr int WGM = BM / 64, WGN = NW / WGM;  // wave grid: 64-row blocks of the tile
    static constexpr int TM = BM / WGM, TN = BN / WGN;   // a wave's block
    static constexpr int WM = TM / 32, WN = TN / 32;     // its 32 x 32 products
    static constexpr int ROWS = BM + BN;                 // rows of a stage
    static constexpr int STAGE = ROWS * BK * 2;          // bytes of a stage
    static constexpr int PER_WAVE = ROWS / 16 / NW;      // load instructions per wave per stage
    // epilogue tile pitch (floats): 16-byte aligned rows; 16 consecutive rows
    // start in distinct 16-byte bank groups
    static constexpr int PITCH = BN + 4;
    static constexpr size_t kStages = (size_t)NS * STAGE, kTile = (size_t)BM / 2 * PITCH * 4;
    static constexpr size_t LDS = kStages > kTile ? kStages : kTile;
    static_assert(ROWS % (16 * NW) == 0, "whole blocks per wave");
    static_assert(WGM * WGN == NW && TM == 64, "wave grid");
    static_assert(LDS <= 160 * 1024, "fits the LDS of a CU");
};

// s_waitcnt vmcnt(n) with the other counters left alone (gfx9 encoding:
// vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
template <int n>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(n >= 0 && n < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Workgroup barrier without the memory fence of __syncthreads, whose release
// half would wait for every outstanding load, the later slices' included.
// The loads a slice needs are waited for explicitly before it; the compiler
// fences keep LDS accesses on their side of the barrier.
__device__ __forceinline__ void barrier_no_fence() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Column tiles of the product: first the routing tiles (whole heads of K
// columns, 256 / K heads each), then for each projection its rows of
// H*2N in tiles of 256.  All scalar.
struct ColTile {
    int kind;   // -1: routing; else the projection's index
    int r0;     // first weight row of the tile
    int ncol;   // valid columns
    int h0, nh; // routing: first head, heads
};

__device__ __forceinline__ ColTile col_tile(const ProjectArgs& a, int nt, int BN) {
    ColTile c;
    const int hpb = a.S ? BN / a.K : 1;
    const int NTr = a.S ? (a.H + hpb - 1) / hpb : 0;
    if (nt < NTr) {
        c.kind = -1;
        c.h0 = nt * hpb;
        c.nh = min(hpb, a.H - c.h0);
        c.r0 = c.h0 * a.K;
        c.ncol = c.nh * a.K;
    } else {
        const int R = 2 * a.H * a.N, NTp = (R + BN - 1) / BN;
        const int j = nt - NTr;
        c.kind = j / NTp;
        c.r0 = (j - c.kind * NTp) * BN;
        c.ncol = min(BN, R - c.r0);
        c.h0 = c.nh = 0;
    }
    return c;
}

__device__ __forceinline__ int col_tiles(const ProjectArgs& a, int BN) {
    const int hpb = a.S ? BN / a.K : 1;
    const int NTr = a.S ? (a.H + hpb - 1) / hpb : 0;
    const int R = 2 * a.H * a.N;
    return NTr + a.nproj * ((R + BN - 1) / BN);
}

// D = sigmoid(m) exp(i p): the diagonal generator of one entry from its two
// projected values (magnitude logit m, phase p).  Which of its two forms gives
// an entry depends on that entry alone, so a token's D has the same bits in
// every kernel and beside any neighbours.
//
// |m| < kGenMag and |p| < kGenPhase (NaN included), in straight-line code: a
// kernel with 256 accumulators cannot afford sincosf's branch for large
// arguments in its epilogue.  exp(-m) = 2^t (1 + v), t - v log2(e) = -m log2(e)
// with log2(e) in two parts; the reciprocal r + rl of 1 + exp(-m) by the
// hardware's r0 and one Newton step on the unrounded sum (1 - r0 is exact for
// r0 >= 1/2), its rounding rl kept for the products; the phase reduced by
// multiples k of pi/2 in three parts (Cody-Waite; k < 2^13: the first
// difference is exact), k rounded by adding 1.5 * 2^23 so that its low bits
// are the quadrant; sin and cos by polynomials fitted for the least largest
// relative error on [-pi/4, pi/4] (6e-9 and 7e-10 with the coefficients
// rounded, below fp32 rounding).
// Error of D relative to |D| against 64 bits, 2^24 samples each, beside
// 1 / (1 + expf(-m)) with sincosf: m, p normal: largest 1.6e-7 (2.0e-7), root
// mean square 4.0e-8 (5.3e-8); m in [-79, 0]: 1.7e-7 (2.1e-7); |p| < 8191:
// 1.7e-7 (1.9e-7); 50 vector instructions (160).
constexpr float kGenMag = 80.f, kGenPhase = 8192.f;
__device__ __forceinline__ float2 diag_gen_small(float m, float p) {
    const float t = m * -0x1.715476p+0f;
    const float u = fmaf(m, -0x1.4ae0cp-26f, fmaf(m, -0x1.715476p+0f, -t));
    const float e = __builtin_amdgcn_exp2f(t), v = u * 0x1.62e430p-1f;
    const float r0 = __builtin_amdgcn_rcpf(1.f + e);
    const float d = fmaf(-(r0 * e), v, fmaf(-r0, e, 1.f - r0));
    const float r = fmaf(d, r0, r0), rl = fmaf(d, r0, r0 - r);
    const float kb = fmaf(p, 0x1.45f306p-1f, 0x1.8p23f), k = kb - 0x1.8p23f;
    float x = fmaf(-k, 0x1.921fb6p+0f, p);
    x = fmaf(k, 0x1.777a5cp-25f, x);
    x = fmaf(k, 0x1.ee59dap-50f, x);
    const float x2 = x * x;
    const float s = fmaf(x * x2, fmaf(x2, fmaf(x2, -0x1.994e5cp-13f, 0x1.11076p-7f), -0x1.555546p-3f), x);
    const float c = fmaf(x2, fmaf(x2, fmaf(x2, fmaf(x2, 0x1.9a020ap-16f, -0x1.6c0c8ap-10f), 0x1.55554ap-5f), -0.5f),
                         1.f);
    const uint32_t q = __float_as_uint(kb);
    const uint32_t flip_s = (q & 2) << 30, flip_c = ((q + 1) & 2) << 30;
    const float ss = __uint_as_float(__float_as_uint(q & 1 ? c : s) ^ flip_s);
    const float cc = __uint_as_float(__float_as_uint(q & 1 ? s : c) ^ flip_c);
    return make_float2(fmaf(r, cc, rl * cc), fmaf(r, ss, rl * ss));
}

__device__ __forceinline__ float2 diag_gen(float m, float p) {
    if (!(fabsf(m) >= kGenMag || fabsf(p) >= kGenPhase)) return diag_gen_small(m, p);
    const float r = 1.f / (1.f + expf(-m));
    float s, c;
    sincosf(p, &s, &c);
    return make_float2(r * c, r * s);
}

template <int BM>
__global__ __launch_bounds__(512) void k_project_dma(ProjectArgs a) {
    using C = RouteDma<BM>;
    constexpr int NT_ = C::NW * 64;
    extern __shared__ __align__(16) unsigned char lds[];
    // wave-uniform in a scalar register: the load instructions' LDS base and
    // descriptor depend on it
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = wv / C::WGN, wn = wv % C::WGN;
    const int NT = col_tiles(a, C::BN), MT = (a.T + BM - 1) / BM;
    const int total = NT * MT;
    int t = blockIdx.x;
    if (total % 8 == 0) t = (t % 8) * (total / 8) + t / 8;
    const int nt = t % NT, mt = t / NT;
    const ColTile ct = col_tile(a, nt, C::BN);
    const int ncol = ct.ncol;
    const int m0 = mt * BM;
    const int HK = a.H * a.K;
    const int R = 2 * a.H * a.N;

    // this lane's byte offset of each of its load instructions: row
    // (wv * PER_WAVE + i) * 16 + lane % 16 of the stage, chunk lane / 16
    const uint32_t row_bytes = (uint32_t)a.Dm * 2;
    const __amdgpu_buffer_rsrc_t ru = row_block(a.u, (uint32_t)a.T * row_bytes);
    const __amdgpu_buffer_rsrc_t rs =
        ct.kind < 0 ? row_block(a.S, (uint32_t)HK * row_bytes) : row_block(a.W[ct.kind], (uint32_t)R * row_bytes);
    uint32_t voff[C::PER_WAVE];
#pragma unroll
    for (int i = 0; i < C::PER_WAVE; ++i) {
        const int row = (wv * C::PER_WAVE + i) * 16 + (lane & 15);
        const uint32_t r = row < BM ? (uint32_t)(m0 + row) : (uint32_t)(ct.r0 + row - BM);
        voff[i] = r * row_bytes + 16u * (uint32_t)(lane >> 4);
    }
    auto issue = [&](int s) {
        unsigned char* st = lds + (s % C::NS) * C::STAGE;
        const uint32_t so = (uint32_t)s * C::BK * 2;
#pragma unroll
        for (int i = 0; i < C::PER_WAVE; ++i)
            load_lds16((wv * C::PER_WAVE + i) * 16 >= BM ? rs : ru, st + (wv * C::PER_WAVE + i) * 1024, voff[i], so);
    };

    f32x16 acc[C::WM][C::WN];
#pragma unroll
    for (int i = 0; i < C::WM; ++i)
#pragma unroll
        for (int j = 0; j < C::WN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int c0 = wn * C::TN;     // this wave's first column of the tile
    const bool work = c0 < ncol;  // a wave past the tile's columns multiplies zeros and stores nothing
    const int ra = wm * C::TM + (lane & 31);  // operand rows: A tile i at ra + 32 i
    const int rb = BM + c0 + (lane & 31);     // B tile j at rb + 32 j
    auto off = [](int r, int c) { return (r >> 4) * 1024 + c * 256 + (r & 15) * 16; };
    // every operand read of a slice is issued before its first product, so
    // the reads of the second half of the slice overlap the products of the first
    auto compute = [&](int s) {
        const unsigned char* st = lds + (s % C::NS) * C::STAGE;
        bf16x8 A[2][C::WM], B[2][C::WN];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int c = 2 * kk + (lane >> 5);
#pragma unroll
            for (int i = 0; i < C::WM; ++i) A[kk][i] = *reinterpret_cast<const bf16x8*>(st + off(ra + 32 * i, c));
#pragma unroll
            for (int j = 0; j < C::WN; ++j) B[kk][j] = *reinterpret_cast<const bf16x8*>(st + off(rb + 32 * j, c));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < C::WM; ++i)
#pragma unroll
                for (int j = 0; j < C::WN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[kk][i], B[kk][j], acc[i][j], 0, 0, 0);
    };

    const int nsl = a.Dm / C::BK;
#pragma unroll
    for (int s = 0; s < C::NS - 1; ++s)
        if (s < nsl) issue(s);
    for (int s = 0; s < nsl; ++s) {
        // this wave's loads of slice s are done once at most the later issued slices are outstanding
        const int ahead = min(C::NS - 2, nsl - 1 - s);
        if (ahead >= 2) wait_vmcnt<2 * C::PER_WAVE>();
        else if (ahead == 1) wait_vmcnt<C::PER_WAVE>();
        else wait_vmcnt<0>();
        barrier_no_fence();  // every wave's slice s is in LDS; every wave is done with slice s-1
        if (s + C::NS - 1 < nsl) issue(s + C::NS - 1);  // into slice s-1's stage
        compute(s);
    }
    __syncthreads();  // the stages are free for the epilogue tile

    float* tile = reinterpret_cast<float*>(lds);
    constexpr int HALF = BM / 2;
    // 16-byte logits stores and argmax reads when K % 4 == 0 (then every head,
    // every tile and every output row starts on a 16-byte boundary)
    const bool vec = a.K % 4 == 0;
    for (int half = 0; half < 2; ++half) {
        if (half) __syncthreads();  // the first half's readers are done
        const int rlo = wm * C::TM - half * HALF;  // this wave's first row within the half
        if (rlo >= 0 && rlo < HALF && work) {
#pragma unroll
            for (int i = 0; i < C::WM; ++i)
#pragma unroll
                for (int j = 0; j < C::WN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        tile[(rlo + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * C::PITCH + c0 + 32 * j +
                             (lane & 31)] = acc[i][j][r];
        }
        __syncthreads();
        const int mb = m0 + half * HALF;
        const int nm = max(0, min(HALF, a.T - mb));
        if (ct.kind >= 0) {
            // a projection: rows of [T, H*2N] floats; R, r0 and ncol are
            // multiples of 4 (2N >= 16), so every row piece is 16-byte aligned
            float* orow = a.out[ct.kind] + (size_t)mb * R + ct.r0;
            const int nq = ncol / 4;
            const bool gen = a.kind[ct.kind] == kProjGen;
            for (int e = threadIdx.x; e < nm * nq; e += NT_) {
                const int m = e / nq, q = e - m * nq;
                float4 v = *reinterpret_cast<const float4*>(tile + m * C::PITCH + 4 * q);
                if (gen) {
                    const float2 d0 = diag_gen(v.x, v.y), d1 = diag_gen(v.z, v.w);
                    v = make_float4(d0.x, d0.y, d1.x, d1.y);
                }
                *reinterpret_cast<float4*>(orow + (size_t)m * R + 4 * q) = v;
            }
            continue;
        }
        float* lrow = a.logits ? a.logits + (size_t)mb * HK + (size_t)ct.h0 * a.K : nullptr;  // row mb, first column
        if (vec) {
            const int nq = ncol / 4;
            if (lrow)
                for (int e = threadIdx.x; e < nm * nq; e += NT_) {
                    const int m = e / nq, q = e - m * nq;
                    *reinterpret_cast<float4*>(lrow + (size_t)m * HK + 4 * q) =
                        *reinterpret_cast<const float4*>(tile + m * C::PITCH + 4 * q);
                }
        } else if (lrow) {
            for (int e = threadIdx.x; e < nm * ncol; e += NT_) {
                const int m = e / ncol, c = e - m * ncol;
                lrow[(size_t)m * HK + c] = tile[m * C::PITCH + c];
            }
        }
        // first maximal index per (token, head); neighbouring lanes take
        // neighbouring tokens
        for (int e = threadIdx.x; e < HALF * ct.nh; e += NT_) {
            const int m = e % HALF, hh = e / HALF;
            if (m >= nm) continue;
            const float* v = tile + m * C::PITCH + hh * a.K;
            int best = 0;
            float bv = v[0];
            if (vec) {
                for (int q = 0; q < a.K / 4; ++q) {
                    const float4 x = reinterpret_cast<const float4*>(v)[q];
                    if (x.x > bv) bv = x.x, best = 4 * q;
                    if (x.y > bv) bv = x.y, best = 4 * q + 1;
                    if (x.z > bv) bv = x.z, best = 4 * q + 2;
                    if (x.w > bv) bv = x.w, best = 4 * q + 3;
                }
            } else {
                for (int k = 1; k < a.K; ++k)
                    if (v[k] > bv) bv = v[k], best = k;
            }
            a.idx[(size_t)(mb + m) * a.H + ct.h0 + hh] = best;
        }
    }
}

// ------------------------------------------------------------------ k_project_wide
// The same product for problems that fill the chip with 256 x 256 tiles and
// are mostly projections.  Four waves, one per SIMD, each 128 x 128 with its
// 256 accumulators in AGPRs: per slice of 64 the operands cost 128 KB of LDS
// reads a workgroup against 192 KB with eight waves of 128 x 64.  Slices come
// as whole 128-byte lines (half lines reach half the L2 rate) through a ring of
// five 32 KB units, so that one and a half slices are in flight while one is
// multiplied; one barrier per 64 matrix instructions of a wave, every other
// instruction of the slice set between them.  The workgroups are persistent
// and run on into the next tile's slices: its loads are in flight during the
// epilogue, which writes (re, im) pairs straight from the accumulators (the
// weights' rows are permuted in LDS so that a pair's two columns fall to one
// lane) without staging or waiting.
//
// Bound: the matrix cores at the clock that the card leaves them.  At 32768
// tokens, d 4096, 26624 columns a launch takes 1.0e7 cycles (1.76 GHz), the
// matrix cores are busy for 68% of them and the waves wait for 16%; no LDS bank
// conflicts; 10.7 GB fetched (u and the weights are 0.5 GB) and 3.2 GB written.
// At d 1024, 6400 columns 45% and 16%.  Measured against eight waves with slices
// of 32 (k_project_dma<256>), in turn on one box: 8068 -> 5792 us (1234 TFLOP/s)
// and 625 -> 473 us (908 TFLOP/s); the vendor library's plain bf16 products with
// bf16 outputs of these sizes take 4620 and 354 us.  Without the L2 prefetch
// the former takes 5.5% more, the latter 1% less, d 64 3% less.
struct WideProj {
    static constexpr int BM = 256, BN = 256, BK = 64;
    static constexpr int ROWB = BK * 2;           // bytes of a row's slice: one 128-byte line
    static constexpr int UNIT = BM * ROWB;        // a ring unit: 256 rows of u or of the weights, 32 KB
    static constexpr int RING = 5;                // units; slice s of u is unit 2s % 5, of the weights (2s + 1) % 5
    static constexpr int PER_WAVE = BM / 8 / 2;   // loads (8 rows each) per wave per slice
    static constexpr int GM = 8;                  // token tiles of a group (see tile_at)
    static constexpr size_t LDS = (size_t)RING * UNIT;
    static_assert(BM == BN && LDS <= 160 * 1024, "fits the LDS of a CU");
};

// 8 bytes at byte offset voff of the buffer, which no later read of this
// kernel wants: kept out of the L2's way.
__device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, uint32_t voff, float2 v) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(v.x), __float_as_uint(v.y)}, r, voff, 0, kLoadStream);
}

// row_block of wave-uniform values that were formed in vector registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_block(const void* base, uint32_t bytes) {
    const uint64_t b = reinterpret_cast<uint64_t>(base);
    return row_block(reinterpret_cast<const void*>((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32 |
                                                   (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b)),
                     __builtin_amdgcn_readfirstlane(bytes));
}

// A tile of the product: 256 tokens x 256 columns, the columns as two halves
// of up to 128 (one per wave column).  Routing halves hold whole heads when
// K <= 128; a larger head spans both halves of its tile.
struct WideTile {
    int m0;      // first token
    int kind;    // -1: routing; else the projection's index
    int r0;      // first weight row of half 0
    int nt;      // column tile
    int hc;      // weight rows of a full half: half 1 starts at r0 + hc
    int rows;    // rows of the weight matrix
    int h0;      // routing: first head of half 0
};

__device__ __forceinline__ int wide_hph(int K) { return K <= 128 ? 128 / K : 1; }  // heads per half (K > 128: per tile)

__host__ __device__ inline int wide_col_tiles(int H, int K, int N, bool route, int nproj) {
    const int per = K <= 128 ? 2 * (128 / K) : 1;
    return (route ? (H + per - 1) / per : 0) + nproj * ((2 * H * N + 255) / 256);
}

__device__ __forceinline__ WideTile wide_tile(const ProjectArgs& a, int nt, int mt) {
    WideTile t;
    t.m0 = mt * WideProj::BM;
    t.nt = nt;
    const int hph = wide_hph(a.K), per = a.K <= 128 ? 2 * hph : 1;
    const int NTr = a.S ? (a.H + per - 1) / per : 0;
    if (nt < NTr) {
        t.kind = -1;
        t.h0 = nt * per;
        t.r0 = t.h0 * a.K;
        t.hc = a.K <= 128 ? hph * a.K : 128;
        t.rows = a.H * a.K;
    } else {
        const int R = 2 * a.H * a.N, NTp = (R + 255) / 256, j = nt - NTr;
        t.kind = j / NTp;
        t.r0 = (j - t.kind * NTp) * 256;
        t.hc = 128;
        t.rows = R;
        t.h0 = 0;
    }
    return t;
}

__global__ __launch_bounds__(256, 1) void k_project_wide(ProjectArgs a) {
    using C = WideProj;
    extern __shared__ __align__(16) unsigned char lds[];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = wv >> 1, wn = wv & 1;
    const int l32 = lane & 31, hf = lane >> 5;
    const int HK = a.H * a.K, R = 2 * a.H * a.N;
    const int NT = wide_col_tiles(a.H, a.K, a.N, a.S != nullptr, a.nproj), MT = (a.T + C::BM - 1) / C::BM;
    const int total = NT * MT;
    // this workgroup's tiles: every (gridDim / 8)-th of its XCD's range
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, nslot = gridDim.x >> 3;
    const int lo = (int)((long long)total * xcd / 8), hi = (int)((long long)total * (xcd + 1) / 8);
    int tc = lo + slot;  // tile being multiplied
    if (tc >= hi) return;
    const int nsl = (a.Dm + C::BK - 1) / C::BK;
    const bool half_tail = a.Dm % C::BK != 0;  // Dm is a multiple of 32: the last slice has two of its four steps

    auto tile_at = [&](int t) {
        const int per = C::GM * NT, g = t / per, rem = t - g * per;
        const int gm = min(C::GM, MT - g * C::GM);
        const int nt = rem / gm;
        return wide_tile(a, nt, g * C::GM + rem - nt * gm);
    };

    // ---- loads: waves 0, 1 bring a slice's 256 rows of u, waves 2, 3 those of
    // the weights, 8 rows of 128 bytes an instruction.  Place r's 16-byte chunk c
    // lies at chunk position c ^ swz(r): any 8 (16) consecutive rows at one
    // chunk fall on distinct banks of 32 (64).
    const uint32_t row_bytes = (uint32_t)a.Dm * 2;
    int tl = tc;             // tile of the next slice to load
    int ls = 0;              // that slice
    int lunit = wv < 2 ? 0 : 1;  // the ring unit it goes to
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t voff[C::PER_WAVE];
    // past the last tile the descriptor is empty: the loads go on, as zeros
    auto point = [&](int t) {
        int ln = lane;
        asm volatile("" : "+v"(ln));  // recomputed here, not kept in registers across the products
        if (t >= hi) {
            rsrc = row_block(a.u, 0);
            return;
        }
        const WideTile w = tile_at(t);
        const bool tok = wv < 2;
        const uint16_t* base = tok ? a.u : w.kind < 0 ? a.S : a.W[w.kind];
        const uint32_t rows = (uint32_t)(tok ? a.T : w.rows);
        const int first = tok ? w.m0 + (wv & 1) * 128 : w.r0 + (wv & 1) * w.hc;
        rsrc = row_block(base, rows * row_bytes);
        // place 8 i + ln / 8 of the wave's 128 holds row 8 i + ln / 8 of u; of the
        // weights, places 64 g + 32 e + l hold row 64 g + 2 l + e
        const uint32_t at = (uint32_t)first * row_bytes + (uint32_t)((ln >> 3) << (tok ? 0 : 1)) * row_bytes;
        const uint32_t last = (rows - 1) * row_bytes;
#pragma unroll
        for (int i = 0; i < C::PER_WAVE; ++i) {
            const int wr = 64 * (i >> 3) + 16 * (i & 3) + (i >> 2 & 1);
            voff[i] = min(at + (uint32_t)(tok ? 8 * i : wr) * row_bytes, last) +
                      16u * (uint32_t)((ln & 7) ^ ((ln >> 3) & 7) ^ (i & 1));
        }
    };
    // a half tail slice holds 64 bytes of each row: its upper chunks start past
    // every descriptor (buffers below 2 GiB) and arrive as zeros
    const uint32_t gone = ((lane & 7) ^ (lane >> 3)) & 4 ? 0x80000000u : 0u;
    uint32_t skip = half_tail && nsl == 1 ? gone : 0u;
    auto issue = [&](int i) {
        load_lds16(rsrc, lds + lunit * C::UNIT + ((wv & 1) * C::PER_WAVE + i) * 1024, voff[i] | skip,
                   (uint32_t)ls * C::ROWB);
    };
    auto next_unit = [](int u) { return u >= C::RING - 2 ? u - (C::RING - 2) : u + 2; };
    auto advance = [&]() {
        lunit = next_unit(lunit);
        if (tl < hi) ++ls;
        if (ls == nsl) {
            ls = 0;
            tl += nslot;
            point(tl);
        }
        skip = half_tail && ls == nsl - 1 ? gone : 0u;
    };
    auto issue_all = [&]() {
#pragma unroll
        for (int i = 0; i < C::PER_WAVE; ++i) issue(i);
        advance();
    };

    // ---- L2 prefetch: the tiles in flight on an XCD share their rows (GM token
    // tiles x 32 / GM column tiles), so each workgroup touches a share of its
    // tile's lines kAhead slices before they are loaded: waves 0, 1 a quarter of
    // the tokens' lines, waves 2, 3 an eighth of the weights'.  One load a slice.
    constexpr int kAhead = 3;
    int pt = tl, ps = 0;
    __amdgpu_buffer_rsrc_t prsrc;
    uint32_t pvoff;
    auto ppoint = [&](int t) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        prsrc = row_block(a.u, 0);
        pvoff = 0;
        if (t >= hi) return;
        const WideTile w = tile_at(t);
        const bool tok = wv < 2;
        const uint16_t* base = tok ? a.u : w.kind < 0 ? a.S : a.W[w.kind];
        const uint32_t rows = (uint32_t)(tok ? a.T : w.rows);
        const int rr = tok ? 64 * (w.nt & 3) + 32 * (wv & 1) + (ln & 31)
                           : 32 * (w.m0 / C::BM & 7) + 16 * (wv & 1) + (ln & 15);
        const int first = tok ? w.m0 + rr : rr < 128 ? w.r0 + rr : w.r0 + w.hc + rr - 128;
        prsrc = row_block(base, rows * row_bytes);
        pvoff = min((uint32_t)first * row_bytes, (rows - 1) * row_bytes);
    };
    uint32_t pf = 0;
    auto padvance = [&]() {
        if (pt < hi && ++ps == nsl) {
            ps = 0;
            pt += nslot;
            ppoint(pt);
        }
    };

    // ---- operand reads: wave (wm, wn) multiplies tokens 128 wm .. and columns
    // 128 wn ..; a lane's columns of products 2jj and 2jj + 1 are the pair
    // 64 jj + 2 l32, + 1 (real and imaginary part of one entry)
    const int swz = (l32 & 7) ^ ((l32 >> 3) & 1);
    uint32_t xu[4], xw[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        xu[kk] = (uint32_t)(wm * 128 + l32) * C::ROWB + 16u * (uint32_t)((2 * kk + hf) ^ swz);
        xw[kk] = (uint32_t)(wn * 128 + l32) * C::ROWB + 16u * (uint32_t)((2 * kk + hf) ^ swz);
    }
    struct Frag {
        bf16x8 u[4], w[4];
    } f[2];
    auto rd_u = [&](int unit, int kk, int i) {
        return *reinterpret_cast<const bf16x8*>(lds + unit * C::UNIT + xu[kk] + 32 * i * C::ROWB);
    };
    auto rd_w = [&](int unit, int kk, int j) {
        return *reinterpret_cast<const bf16x8*>(lds + unit * C::UNIT + xw[kk] + 32 * j * C::ROWB);
    };
    // acc[i][j]: lane = column, register r = token 32 i + 8 (r / 4) + 4 hf + r % 4
    f32x16 acc[4][4];
    // one step of 16: 16 products on fragment set cur and, between them, the
    // next step's eight operand reads and half (1: first, 2: second) of a
    // slice's loads; the second half moves the cursors on
    auto step = [&](auto cur_, int uu, int uw, int rkk, auto loads_) {
        constexpr int cur = decltype(cur_)::value;
        constexpr int LOADS = decltype(loads_)::value;
        Frag& n = f[cur ^ 1];
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int i = m >> 2, j = m & 3;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[cur].u[i], f[cur].w[j], acc[i][j], 0, 0, 0);
            if (m == 0) n.u[0] = rd_u(uu, rkk, 0);
            if (m == 1) n.w[0] = rd_w(uw, rkk, 0);
            if (m == 2) n.w[1] = rd_w(uw, rkk, 1);
            if (m == 3) n.w[2] = rd_w(uw, rkk, 2);
            if (m == 4) n.w[3] = rd_w(uw, rkk, 3);
            if (m == 5) n.u[1] = rd_u(uu, rkk, 1);
            if (m == 7) n.u[2] = rd_u(uu, rkk, 2);
            if (m == 9) n.u[3] = rd_u(uu, rkk, 3);
            if constexpr (LOADS == 1)
                if (m % 2 == 0) issue(m / 2);
            if constexpr (LOADS == 2) {
                if (m < 8) issue(m + C::PER_WAVE / 2);
                if (m == 9) {
                    asm volatile("" ::"v"(pf));  // a slice old
                    pf = __builtin_amdgcn_raw_buffer_load_b32(prsrc, pvoff, (uint32_t)ps * C::ROWB, 0);
                }
                if (m == 11) advance();
                if (m == 13) padvance();
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using c0 = std::integral_constant<int, 0>;
    using c1 = std::integral_constant<int, 1>;
    using c2 = std::integral_constant<int, 2>;

    // ---- prologue: slice 0 (and 1 of u) of the flattened sequence, then the
    // first half of the next
    auto issue_half = [&]() {
#pragma unroll
        for (int i = 0; i < C::PER_WAVE / 2; ++i) issue(i);
    };
    point(tl);
    issue_all();
    if (wv < 2) {
        issue_all();
        issue_half();
        wait_vmcnt<3 * C::PER_WAVE / 2>();
    } else {
        issue_half();
        wait_vmcnt<C::PER_WAVE / 2>();
    }
    ppoint(pt);
    for (int i = 0; i < 2 + kAhead; ++i) padvance();
    barrier_no_fence();
    int uu = 0, uw = 1;  // ring units of the slice being multiplied
    f[0].u[0] = rd_u(uu, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) f[0].w[j] = rd_w(uw, 0, j);
#pragma unroll
    for (int i = 1; i < 4; ++i) f[0].u[i] = rd_u(uu, 0, i);

    bool stores = false;  // at least 63 stores follow the last loads issued
    for (;;) {
        const WideTile w = tile_at(tc);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        // every read of this slice's units has returned and the next slice has
        // arrived, for every wave: the units may be loaded again.  Waves 0, 1
        // may have the u slice after the next in flight (and with 63 stores
        // after it, the next has been answered: answers come in order); the last
        // prefetch may be in flight.
        auto turn = [&]() {
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
            if (wv >= 2) wait_vmcnt<1>();
            else if (!stores) wait_vmcnt<C::PER_WAVE + 1>();
            stores = false;
            barrier_no_fence();
        };
        // the slice's last step: the next slice's first reads, and the loads of
        // a later one into the units just finished
        int done_w = 0;  // the unit that waves 0, 1 are loading u into
        auto last = [&](auto cur) {
            done_w = uw;
            const int nu = next_unit(uu), nw = next_unit(uw);
            step(cur, nu, nw, 0, c1{});
            uu = nu;
            uw = nw;
        };
        for (int s = 0; s < nsl; ++s) {
            step(c0{}, uu, uw, 1, c2{});
            step(c1{}, uu, uw, 2, c0{});
            step(c0{}, uu, uw, 3, c0{});
            turn();
            last(c1{});
        }
        // ---- epilogue.  Lane-dependent addresses are formed here from an opaque
        // copy of the lane, not kept in registers across the products.
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int l32 = ln & 31, hf = ln >> 5;
        const int tb = w.m0 + wm * 128;             // first token of this wave's block
        const int nt = max(0, min(128, a.T - tb));  // its tokens
        const int cr = w.r0 + wn * w.hc;            // its first weight row
        if (w.kind >= 0) {
            // a projection: rows of [T, H*2N] floats, a lane's pair of columns
            // one 8-byte store (32 lanes: 256 contiguous bytes of a row), never
            // waited for.  The descriptor ends after the block's last token and
            // a lane past the last column starts beyond it: those stores drop.
            const int ncol = wide_cols(R, cr);
            const bool gen = a.kind[w.kind] == kProjGen;
            float* out = a.out[w.kind] + (size_t)tb * R + cr;
            const __amdgpu_buffer_rsrc_t ro = uniform_block(out, wide_block_bytes(nt, R, ncol));
            uint32_t at[2];
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
                at[jj] = wide_pair_offset(4 * hf, 64 * jj + 2 * l32, R, ncol);
            float most = 0.f;  // largest |m| / kGenMag and |p| / kGenPhase seen
            auto emit = [&](auto f) {
                uint32_t v0 = at[0], v1 = at[1], step = (uint32_t)R * 4;
                asm volatile("" : "+s"(step));  // row offsets formed here, not kept across the products
                if (nt == 0 || ncol == 0) return;  // nothing of this wave's
                auto rows = [&](auto both) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            store_pair(ro, v0, f(acc[i][0][r], acc[i][1][r]));
                            if constexpr (both) store_pair(ro, v1, f(acc[i][2][r], acc[i][3][r]));
                            v0 += (r & 3) == 3 ? 5 * step : step;  // token 32 i + 8 (r / 4) + r % 4 + 4 hf
                            v1 += (r & 3) == 3 ? 5 * step : step;
                            __builtin_amdgcn_sched_barrier(0);
                        }
                };
                if (ncol > 64) rows(std::true_type{});
                else rows(std::false_type{});
            };
            if (gen)
                emit([&](float m, float p) {
                    most = fmaxf(most, fmaxf(fabsf(m) * (1.f / kGenMag), fabsf(p) * (1.f / kGenPhase)));
                    return diag_gen_small(m, p);
                });
            const bool large = __any(most >= 1.f);  // NaN passes through diag_gen_small unharmed
            if (!gen || large) emit([](float m, float p) { return make_float2(m, p); });
            if (large)  // entry by entry, on the values just stored, each by its own lane
#pragma unroll 1
                for (int e = 0; e < 128; ++e) {
                    const int t = 32 * (e >> 5) + 8 * (e >> 3 & 3) + 4 * hf + (e >> 1 & 3), c = 64 * (e & 1) + 2 * l32;
                    if (t >= nt || c >= ncol) continue;
                    float2* o = reinterpret_cast<float2*>(out + (size_t)t * R + c);
                    const float2 v = *o;
                    *o = diag_gen(v.x, v.y);
                }
            stores = nt == 128 && ncol == 128;
        } else {
            // routing: 32 tokens x 64 columns at a time through a staging area
            // of this wave in the ring unit that half of a later u slice went to
            // (loaded once more afterwards)
            wait_vmcnt<0>();
            barrier_no_fence();
            unsigned char* stg = lds + done_w * C::UNIT + wv * (C::UNIT / 4);
            const int hd0 = a.K <= 128 ? w.h0 + wn * wide_hph(a.K) : w.h0;  // this half's first head
            const int ncol = a.K <= 128 ? min(wide_hph(a.K), a.H - hd0) * a.K : wn == 0 ? 128 : a.K - 128;
            const bool fresh = a.K <= 128 || wn == 0;  // else the second half of a head: nothing chosen yet
            const int rq = ln >> 4, q = ln & 15;       // rows rq, rq + 4, ...; columns 4q .. 4q + 3
            // 16-byte chunk q of a staged row lies at chunk position q ^ (row % 16)
            float bv[4];
            int best[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int k = 0, hd = hd0;
                bv[i] = -INFINITY, best[i] = -1;
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                    const int left = ncol - 64 * jj;
                    if (left <= 0) continue;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int t = 8 * (r >> 2) + 4 * hf + (r & 3);
                        *reinterpret_cast<float2*>(stg + t * 256 + 16 * ((l32 >> 1) ^ (t & 15)) + 8 * (l32 & 1)) =
                            make_float2(acc[i][2 * jj][r], acc[i][2 * jj + 1][r]);
                    }
                    auto piece = [&](int row, int q) {
                        return *reinterpret_cast<const float4*>(stg + row * 256 + 16 * (q ^ (row & 15)));
                    };
                    float* lg = a.logits + (size_t)(tb + 32 * i + rq) * HK + cr + 64 * jj + 4 * q;
                    if (a.logits && a.K % 4 == 0) {  // whole pieces: eight reads, then their stores
                        float4 v[8];
#pragma unroll
                        for (int it = 0; it < 8; ++it) v[it] = piece(4 * it + rq, q);
#pragma unroll
                        for (int it = 0; it < 8; ++it)
                            if (32 * i + 4 * it + rq < nt && 4 * q < left)
                                *reinterpret_cast<float4*>(lg + (size_t)(4 * it) * HK) = v[it];
                    } else if (a.logits) {
#pragma unroll 1
                        for (int it = 0; it < 8; ++it) {
                            const float4 v = piece(4 * it + rq, q);
                            const int c = 64 * jj + 4 * q;
                            float* o = lg + (size_t)(4 * it) * HK;
                            if (32 * i + 4 * it + rq >= nt) continue;
                            if (c < ncol) o[0] = v.x;
                            if (c + 1 < ncol) o[1] = v.y;
                            if (c + 2 < ncol) o[2] = v.z;
                            if (c + 3 < ncol) o[3] = v.w;
                        }
                    }
                    // first maximal column of each head, lane = token
                    float4 x = piece(l32, 0);
#pragma unroll 1
                    for (int p = 0; 4 * p < min(left, 64); ++p) {
                        const float4 y = piece(l32, (p + 1) & 15);
                        auto take = [&](float v, bool on) {
                            if (!on) return;
                            if ((fresh && k == 0) || v > bv[i]) bv[i] = v, best[i] = k;
                            if (++k == a.K) {
                                if (hf == 0 && 32 * i + l32 < nt)
                                    a.idx[(size_t)(tb + 32 * i + l32) * a.H + hd] = best[i];
                                k = 0;
                                ++hd;
                            }
                        };
                        take(x.x, true);
                        take(x.y, 4 * p + 1 < left);
                        take(x.z, 4 * p + 2 < left);
                        take(x.w, 4 * p + 3 < left);
                        x = y;
                    }
                }
            }
            if (a.K > 128) {  // the head's other half comes from the neighbouring wave
                if (wn == 1 && hf == 0)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        *reinterpret_cast<float2*>(stg + (32 * i + l32) * 8) =
                            make_float2(bv[i], __int_as_float(best[i]));
                __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
                barrier_no_fence();
                if (wn == 0 && hf == 0)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float2 o =
                            *reinterpret_cast<const float2*>(stg + C::UNIT / 4 + (32 * i + l32) * 8);
                        if (32 * i + l32 < nt)
                            a.idx[(size_t)(tb + 32 * i + l32) * a.H + w.h0] =
                                o.x > bv[i] ? 128 + __float_as_int(o.y) : best[i];
                    }
            }
            __builtin_amdgcn_s_waitcnt(0xc07f);
            barrier_no_fence();
            if (wv < 2) issue_half();
        }
        tc += nslot;
        if (tc >= hi) break;
    }
    wait_vmcnt<0>();  // nothing lands in this LDS after the workgroup ends
}

// ------------------------------------------------------------------ k_project_thin
// The same product for few tokens (one step of generation for a batch), bound
// by reading the weights once: a wave takes 32 weight rows against 32 TB tokens
// over the whole contraction, in the other kernels' order, so a token's outputs
// have the same bits in any call (a near-tie chooses the same map in generation
// as in prefill).  A routing workgroup takes whole heads, up to 128 rows, and
// the launch has as many waves a workgroup as that needs.  A wave streams its
// slices of 64 (whole lines: 16 bytes a lane straight into operand registers
// would touch 64 lines an instruction, which the address unit, not memory,
// paces) through NS LDS stages of its own, no barrier on the way.
// Stages: 8 KB of 32 tokens, 12 KB of 64.  With up to 512 waves (two a CU) 8
// stages, with more 5, so that four fit a CU: fewer leave memory idle (6400
// rows of d 1024, one token: 5.6 us with 8, 6.1 with 5, 8.1 with 3), more stop
// the waves from running at once (769 waves of d 256: 7.5 us with 5, 9.7 with 6).
// 64 tokens: 5, or 3 where four waves must fit.
// Measured (weights not in cache), 128-token tiles -> these: 26624 rows of d
// 4096, one token 85 -> 44 us (5.0 TB/s), 32 tokens 92 -> 51, 64 tokens 100 ->
// 60; 6400 rows of d 1024 23 -> 5.6, 26 -> 7.2 and 30 -> 10.4; 800 rows of d
// 4096, one token 70 -> 10.8, where one wave's chain of products is the time
// (four waves sharing a contraction would take 8.8 there, but in another order).
// With 128 tokens the 128-token tiles are faster (98 us against 114 for the
// first shape), so they take over beyond 64.
template <int TB, int NS_>
struct ThinProj {
    static constexpr int NS = NS_;
    static constexpr int TT = 32 * TB;          // tokens of a workgroup
    static constexpr int STAGE = (1 + TB) * 32 * 128;  // a slice of 32 weight rows and TT tokens
    static constexpr int LOADS = STAGE / 1024;  // load instructions of a slice
    static constexpr int PITCH = 33;            // floats of a result row: 32 columns, padded
    static constexpr int WAVE = NS * STAGE;     // bytes of a wave, its results over its stages
    static_assert(TT * PITCH * 4 <= WAVE && (NS - 1) * LOADS < 64, "results fit; vmcnt range");
};

__host__ __device__ inline int thin_heads(int K) { return K < 32 ? 32 / K : 1; }  // heads of a routing workgroup
// waves of a workgroup: those of a routing workgroup, a power of two
__host__ __device__ inline int thin_waves(int K, bool route) { return !route || K <= 32 ? 1 : K <= 64 ? 2 : 4; }

template <int TB, int NS>
__global__ __launch_bounds__(256) void k_project_thin(ProjectArgs a) {
    using C = ThinProj<TB, NS>;
    extern __shared__ __align__(16) unsigned char lds[];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l32 = lane & 31, hf = lane >> 5;
    const int R = 2 * a.H * a.N, HK = a.H * a.K;
    const int t0 = blockIdx.y * C::TT, nt = min(C::TT, a.T - t0);
    const int hpb = thin_heads(a.K), NTr = a.S ? (a.H + hpb - 1) / hpb : 0;
    const int W = thin_waves(a.K, a.S != nullptr), lg = W >> 1;  // waves (1, 2, 4), their logarithm
    const int cols = 32 * W;                                     // columns of a projection's workgroup
    int kind = -1, r0, ncol, rows;
    if ((int)blockIdx.x < NTr) {
        r0 = blockIdx.x * hpb * a.K;
        rows = HK;
        ncol = min(hpb * a.K, HK - r0);
    } else {
        const int NTp = (R + cols - 1) / cols, j = blockIdx.x - NTr;
        kind = j / NTp;
        r0 = (j - kind * NTp) * cols;
        rows = R;
        ncol = min(cols, R - r0);
    }
    // column c of token t, in the stages of the wave that made it
    auto at = [&](int t, int c) {
        return reinterpret_cast<float*>(lds + (c >> 5) * C::WAVE) + t * C::PITCH + (c & 31);
    };
    if (32 * wv < ncol) {
        // loads and operand reads as in k_project_wide: 8 rows of a line an
        // instruction, chunk c of row r at chunk position c ^ swz(r)
        unsigned char* st = lds + wv * C::WAVE;
        const uint32_t row_bytes = (uint32_t)a.Dm * 2;
        const __amdgpu_buffer_rsrc_t rw = row_block(kind < 0 ? a.S : a.W[kind], (uint32_t)rows * row_bytes);
        const __amdgpu_buffer_rsrc_t ru = row_block(a.u, (uint32_t)a.T * row_bytes);
        uint32_t voff[C::LOADS];
#pragma unroll
        for (int i = 0; i < C::LOADS; ++i) {
            const int p = 8 * (i & 3) + (lane >> 3);
            const int row = i < 4 ? min(r0 + 32 * wv + p, rows - 1) : min(t0 + 32 * (i / 4 - 1) + p, a.T - 1);
            voff[i] = (uint32_t)row * row_bytes + 16u * (uint32_t)((lane & 7) ^ ((lane >> 3) & 7) ^ (i & 1));
        }
        // load instructions from .. to - 1 of slice s.  Of a half slice, the last
        // one of a wave, the upper chunks then start past the (below 2 GiB)
        // descriptors and arrive as zeros.
        const int half = a.Dm % 64 ? a.Dm / 64 : -1;
        auto issue = [&](int s, int g, int from, int to) {
            if (s == half && from == 0) {
#pragma unroll
                for (int i = 0; i < C::LOADS; ++i) voff[i] |= ((lane & 7) ^ (lane >> 3)) & 4 ? 0x80000000u : 0u;
            }
#pragma unroll
            for (int i = 0; i < C::LOADS; ++i)
                if (i >= from && i < to)
                    load_lds16(i < 4 ? rw : ru, st + g * C::STAGE + i * 1024, voff[i], (uint32_t)s * 128);
        };
        f32x16 acc[TB];
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
        const int nsl = (a.Dm + 63) / 64;
        const int swz = (l32 & 7) ^ ((l32 >> 3) & 1);
        struct Frag {
            bf16x8 w[4], u[TB][4];
        } f[2];
        // operands of a slice's 16-wide step kk from stage g
        auto read = [&](Frag& f, int g, int kk) {
            const unsigned char* p = st + g * C::STAGE + l32 * 128 + 16 * ((2 * kk + hf) ^ swz);
            f.w[kk] = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
            for (int b = 0; b < TB; ++b) f.u[b][kk] = *reinterpret_cast<const bf16x8*>(p + (b + 1) * 4096);
        };
        auto multiply = [&](const Frag& f, int kk) {
#pragma unroll
            for (int b = 0; b < TB; ++b)
                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.u[b][kk], f.w[kk], acc[b], 0, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (i < nsl) issue(i, i, 0, C::LOADS);
        if (nsl < NS) wait_vmcnt<0>();
        else wait_vmcnt<(NS - 1) * C::LOADS>();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) read(f[0], 0, kk);
        // slice s is multiplied; between its products, each waiting for the one
        // before, slice s + 1 is read and slice s + NS asked for, into the
        // stage of slice s
        int s = 0, g = 0;
        auto step = [&](const Frag& cur, Frag& next) {
            const int gn = g + 1 == NS ? 0 : g + 1;
            __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): slice s is in registers
            wait_vmcnt<(NS - 2) * C::LOADS>();   // slice s + 1 is in LDS
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                multiply(cur, kk);
                read(next, gn, kk);
                issue(s + NS, g, kk * C::LOADS / 4, (kk + 1) * C::LOADS / 4);
                __builtin_amdgcn_sched_barrier(0);
            }
            g = gn;
            ++s;
        };
        while (s + NS + 1 < nsl) {
            step(f[0], f[1]);
            step(f[1], f[0]);
        }
        if (s + NS < nsl) {
            step(f[0], f[1]);
            f[0] = f[1];
        }
        // the last slices, all asked for
        const int rem = nsl - s;
        auto tail = [&](auto i_, auto&& self) {
            constexpr int i = decltype(i_)::value;
            if constexpr (i + 1 < NS)
                if (i + 1 < rem) {
                    g = g + 1 == NS ? 0 : g + 1;
                    wait_vmcnt<(NS - 2 - i) * C::LOADS>();
                    __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) read(f[(i + 1) & 1], g, kk);
                }
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) multiply(f[i & 1], kk);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i + 1 < NS)
                if (i + 1 < rem) self(std::integral_constant<int, i + 1>{}, self);
        };
        tail(std::integral_constant<int, 0>{}, tail);
        // every load has arrived and every stage has been read: the results may go there
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) *at(32 * b + 8 * (r >> 2) + 4 * hf + (r & 3), 32 * wv + l32) = acc[b][r];
    }
    __syncthreads();

    const int threads = 64 * W;
    if (kind >= 0) {
        const bool gen = a.kind[kind] == kProjGen;
        float* out = a.out[kind] + (size_t)t0 * R + r0;
        for (int e = threadIdx.x; e < nt * cols / 2; e += threads) {
            const int t = e >> lg >> 4, c = 2 * e & (cols - 1);
            if (c >= ncol) continue;
            const float x = *at(t, c), y = *at(t, c + 1);
            *reinterpret_cast<float2*>(out + (size_t)t * R + c) = gen ? diag_gen(x, y) : make_float2(x, y);
        }
        return;
    }
    if (a.logits)
        for (int e = threadIdx.x; e < nt * cols; e += threads) {
            const int t = e >> lg >> 5, c = e & (cols - 1);
            if (c < ncol) a.logits[(size_t)(t0 + t) * HK + r0 + c] = *at(t, c);
        }
    // first maximum of each (token, head): by one lane, neighbouring lanes taking
    // neighbouring tokens, or, of more than 64 columns (one head of 256 threads),
    // by eight lanes, each a run of the columns (17 tokens, K = 100: 19.1 -> 16.3
    // us a call; 64 tokens, K = 40: 7.4 by one lane, 8.9 by eight)
    const int nh = ncol / a.K;
    if (a.K <= 64) {
        for (int e = threadIdx.x; e < C::TT * nh; e += threads) {
            const int t = e % C::TT, c0 = e / C::TT * a.K;
            if (t >= nt) continue;
            int best = 0;
            float bv = *at(t, c0);
#pragma unroll 4
            for (int k = 1; k < a.K; ++k) {
                const float v = *at(t, c0 + k);
                if (v > bv) bv = v, best = k;
            }
            a.idx[(size_t)(t0 + t) * a.H + (r0 + c0) / a.K] = best;
        }
        return;
    }
    const int run = (a.K + 7) / 8, sub = threadIdx.x & 7;
    for (int t = threadIdx.x >> 3; t < C::TT; t += threads / 8) {
        float bv = -INFINITY;
        int best = -1;
        for (int k = sub * run; k < min(a.K, (sub + 1) * run); ++k) {
            const float v = *at(t, k);
            if (k == 0 || v > bv) bv = v, best = k;
        }
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {  // the lower run first: it wins ties
            const float ov = __shfl_xor(bv, d);
            const int ob = __shfl_xor(best, d);
            if (!(sub & d) ? ov > bv : ov >= bv && ob >= 0) bv = ov, best = ob;
        }
        if (t < nt && sub == 0) a.idx[(size_t)(t0 + t) * a.H + r0 / a.K] = best;
    }
}

template <int BM>
hipError_t project_dma_launch(const ProjectArgs& a, hipStream_t st) {
    using C = RouteDma<BM>;
    const int hpb = a.S ? C::BN / a.K : 1;
    const int NT = (a.S ? (a.H + hpb - 1) / hpb : 0) + a.nproj * ((2 * a.H * a.N + C::BN - 1) / C::BN);
    const int MT = (a.T + BM - 1) / BM;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_project_dma<BM>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_project_dma<BM>, dim3((unsigned)(NT * MT)), dim3(C::NW * 64), C::LDS, st, a);
    return hipGetLastError();
}

hipError_t project_wide_launch(const ProjectArgs& a, hipStream_t st) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_project_wide),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)WideProj::LDS);
    if (e != hipSuccess) return e;
    // tokens of one launch: u below 2 GiB (byte offsets leave the top bit free)
    const long long fit = ((1LL << 31) / (2LL * a.Dm) - 256) / 256 * 256;
    for (long long t0 = 0; t0 < a.T; t0 += fit) {
        ProjectArgs p = a;
        p.T = (int)(a.T - t0 < fit ? a.T - t0 : fit);
        p.u += t0 * a.Dm;
        if (p.logits) p.logits += t0 * a.H * a.K;
        if (p.idx) p.idx += t0 * a.H;
        for (int j = 0; j < a.nproj; ++j) p.out[j] += t0 * 2 * a.H * a.N;
        hipLaunchKernelGGL(k_project_wide, dim3(256), dim3(256), WideProj::LDS, st, p);
    }
    return hipGetLastError();
}

template <int TB, int NS>
hipError_t project_thin_run(const ProjectArgs& a, int blocks, int waves, hipStream_t st) {
    using C = ThinProj<TB, NS>;
    // the most any launch of this kernel takes: the same from every thread
    constexpr int kMost = (4 * C::WAVE <= 160 * 1024 ? 4 : 2) * C::WAVE;
    static_assert(kMost <= 160 * 1024, "fits the LDS of a CU");
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_project_thin<TB, NS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMost);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_project_thin<TB, NS>), dim3((unsigned)blocks, (unsigned)((a.T + C::TT - 1) / C::TT)),
                       dim3(64 * waves), waves * C::WAVE, st, a);
    return hipGetLastError();
}

template <int TB>
hipError_t project_thin_launch(const ProjectArgs& a, hipStream_t st) {
    const int hpb = thin_heads(a.K), W = thin_waves(a.K, a.S != nullptr), R = 2 * a.H * a.N;
    const int blocks = (a.S ? (a.H + hpb - 1) / hpb : 0) + a.nproj * ((R + 32 * W - 1) / (32 * W));
    if (TB == 2) return W <= 2 ? project_thin_run<2, 5>(a, blocks, W, st) : project_thin_run<2, 3>(a, blocks, W, st);
    return W <= 2 && blocks * W <= 512 ? project_thin_run<1, 8>(a, blocks, W, st)
                                       : project_thin_run<1, 5>(a, blocks, W, st);
}

hipError_t project_dma(const ProjectArgs& a, hipStream_t st) {
    switch (project_kernel(a.T, a.Dm, a.H, a.K, a.N, a.S != nullptr, a.nproj)) {
        case kProjectThin1: return project_thin_launch<1>(a, st);
        case kProjectThin2: return project_thin_launch<2>(a, st);
        case kProjectDma128: return project_dma_launch<128>(a, st);
        case kProjectDma256: return project_dma_launch<256>(a, st);
        case kProjectWide: break;
    }
    return project_wide_launch(a, st);
}

// pi[h,k,j] = argmax_i M[h,k,i,j].  A workgroup takes 64 columns of one
// matrix (h,k) (loads coalesced over j); its four waves each scan a quarter
// of the rows with eight loads in flight, and wave 0 combines the quarters in
// row order, so the first maximal row wins as in a single pass.
constexpr int kArgCols = 64;
__global__ __launch_bounds__(256) void k_dict_argmax(const float* __restrict__ M, int* __restrict__ pi, int HK,
                                                     int N) {
    __shared__ float sv[4][kArgCols];
    __shared__ int si[4][kArgCols];
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int per = (N + kArgCols - 1) / kArgCols;  // column blocks per matrix
    const int g = blockIdx.x / per;
    const int j = (blockIdx.x - g * per) * kArgCols + lane;
    const bool on = g < HK && j < N;
    const int rows = N / 4;  // N is a power of two >= 8
    const int i0 = part * rows;
    const float* col = M + ((size_t)(on ? g : 0) * N + i0) * N + (on ? j : 0);
    int best = i0;
    float bv = col[0];
#pragma unroll 8
    for (int i = 1; i < rows; ++i) {
        const float v = col[(size_t)i * N];
        if (v > bv) bv = v, best = i0 + i;
    }
    sv[part][lane] = bv;
    si[part][lane] = best;
    __syncthreads();
    if (part == 0 && on) {
#pragma unroll
        for (int q = 1; q < 4; ++q)
            if (sv[q][lane] > bv) bv = sv[q][lane], best = si[q][lane];
        pi[(size_t)g * N + j] = best;
    }
}

}  // namespace

// byte offsets of the direct-load kernel are 32-bit, rows past the end included
bool project_fits(long long T, long long rows, long long Dm) {
    return (T + 256) * Dm * 2 < (1LL << 32) && (rows + 256) * Dm * 2 < (1LL << 32);
}

hipError_t launch_route(const RouteArgs& a, hipStream_t st) {
    if (a.Dm % RouteDma<128>::BK == 0 && project_fits(a.T, (long long)a.H * a.K, a.Dm)) {
        ProjectArgs p = {};
        p.T = a.T;
        p.Dm = a.Dm;
        p.H = a.H;
        p.K = a.K;
        p.N = 8;
        p.u = a.u;
        p.S = a.S;
        p.logits = a.logits;
        p.idx = a.idx;
        p.nproj = 0;
        return project_dma(p, st);
    }
    const int hpb = kRouteTN / a.K;
    dim3 grid((a.T + kRouteTM - 1) / kRouteTM, (a.H + hpb - 1) / hpb);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_route),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRouteLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_route, grid, dim3(256), kRouteLds, st, a);
    return hipGetLastError();
}

hipError_t launch_project(const ProjectArgs& a, hipStream_t st) {
    const long long rows = a.S ? (long long)a.H * a.K : 0;
    if (a.Dm % RouteDma<128>::BK != 0 || !project_fits(a.T, rows > 2LL * a.H * a.N ? rows : 2LL * a.H * a.N, a.Dm))
        return hipErrorInvalidValue;
    return project_dma(a, st);
}

hipError_t launch_dict_argmax(const float* M, int* pi, int HK, int N, hipStream_t st) {
    const int64_t blocks = (int64_t)HK * ((N + kArgCols - 1) / kArgCols);
    hipLaunchKernelGGL(k_dict_argmax, dim3((unsigned)blocks), dim3(256), 0, st, M, pi, HK, N);
    return hipGetLastError();
}

}  // namespace pdssm
