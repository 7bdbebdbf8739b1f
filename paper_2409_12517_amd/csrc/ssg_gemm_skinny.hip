// FP8 contraction of few rows for gfx950: the small batches of the inference form and small public calls.
//
//   C[m,n] = sum_k A[m,k] * B[n,k]      A [M,K], B [N,K] FP8 codes, K contiguous
//
// Bound by HBM where M is small (every byte of B is used once), and by what a compute unit can fetch (about 50 bytes per
// clock) where it is a few hundred.  The tiles of ssg_gemm_tile.h have too few workgroups there: 32 for N = 4096, each
// walking all of K alone.  So
//   - a workgroup owns 16 * MB rows of A and 16 * NB rows of B (SwiGLU form: half of them from W1, half the same rows
//     of W2) and its KW waves divide K among them; their partial sums meet in LDS and are added in a fixed order;
//   - every wave streams its own K range through a ring of its own in LDS, STEPS steps of 128 bytes deep: nothing is
//     shared between waves before the end, so there is no barrier in the loop, only each wave's own waits.  (Fragments
//     loaded straight into registers take 4 times the cycles of the texture path: neighbouring lanes hold different
//     rows, so no two of them share a 64-byte piece.);
//   - v_mfma_f32_16x16x128_f8f6f4: 16 rows of A are no waste, and one instruction consumes a whole step.
#include <algorithm>

#include "ssg_gemm_tile.h"

namespace ssg {


constexpr int kBlockBytes = 16 * BK;          // 16 rows of one K step: two DMA instructions
constexpr int skinny_smem(int MB, int NB, int KW, int STEPS) { return KW * STEPS * (MB + NB) * kBlockBytes; }

// The work of workgroup `block`.
template <int EPI, int AFMT, int MB, int NB, int KW, int STEPS>
__device__ __forceinline__ void gemm_skinny_block(const GemmParams &p, const unsigned block, uint8_t *smem) {
    constexpr bool kDual = EPI == EPI_SWIGLU_Q;
    constexpr int NCOL = kDual ? NB / 2 : NB;                          // 16-column blocks of the result
    constexpr int kStepBytes = (MB + NB) * kBlockBytes, kPitch = 16 * NB + 1;
    static_assert(KW * MB * 16 * kPitch * 4 <= skinny_smem(MB, NB, KW, STEPS), "the partial sums reuse the rings");
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the row blocks that share 16 * NB rows of B run on the same XCD one after the other: B comes into its L2 once
    const int mblocks = (int)((p.M + 16 * MB - 1) / (16 * MB)), idx = (int)(block >> 3);
    const int64_t m0 = (int64_t)(idx % mblocks) * (16 * MB);
    const int64_t n0 = ((int64_t)(idx / mblocks) * 8 + (block & 7)) * (16 * NCOL);
    if (n0 >= p.N) return;
    const int ksteps = (int)((p.K + BK - 1) / BK), per = (ksteps + KW - 1) / KW;
    const int s0 = w * per, n = (s0 + per < ksteps ? per : ksteps - s0);      // this wave's steps; may be 0 or less

    // DMA: instruction j of a step brings rows 8j .. 8j+7 of the MB + NB blocks, a lane 16 bytes; row r's chunk c lies at
    // position c ^ swz(r), so that 16 lanes reading the same chunk of 16 rows meet no bank conflict
    const int lrow = l >> 3;
    uint32_t lane_off[2 * (MB + NB)];
#pragma unroll
    for (int j = 0; j < 2 * (MB + NB); ++j) {
        const int row = 8 * (j & 1) + lrow, ck = ((l & 7) ^ swz(row)) * 16;
        // rows beyond the matrix are clamped: they only feed results that are not stored
        int64_t g;
        if (j < 2 * MB) { g = m0 + 8 * j + lrow; g = g < p.M ? g : p.M - 1; }
        else { g = n0 + ((j / 2 - MB) % NCOL) * 16 + row; g = g < p.N ? g : p.N - 1; }
        lane_off[j] = (uint32_t)(g * p.K) + ck;
    }
    const uint32_t ring = (uint32_t)(uintptr_t)(lds_void_ptr)smem + (uint32_t)w * (STEPS * kStepBytes);
    auto issue = [&](int s, int slot) {
        const int64_t k = (int64_t)(s0 + s) * BK;
        const uint32_t dst = ring + (uint32_t)slot * kStepBytes;
        auto base = [&](int j) { return (j < 2 * MB ? p.A : !kDual || j / 2 - MB < NCOL ? p.B : p.B2) + k; };
        if (k + BK <= p.K) {
#pragma unroll
            for (int j = 0; j < 2 * (MB + NB); ++j) dma16_s(base(j), lane_off[j], dst + j * 1024);
        } else {                                      // ragged last step: zeros past K, a multiple of 16
#pragma unroll
            for (int j = 0; j < 2 * (MB + NB); ++j) {
                const int ck = ((l & 7) ^ swz(8 * (j & 1) + lrow)) * 16;
                dma16(k + ck < p.K ? base(j) + lane_off[j] : reinterpret_cast<const uint8_t *>(&g_zero_chunk), dst + j * 1024);
            }
        }
    };
    uint32_t frag_off[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) frag_off[e] = (uint32_t)((l & 15) * BK + ((((l >> 4) * 2 + e) ^ swz(l & 15)) << 4));
    v4f acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

#pragma unroll
    for (int s = 0; s < STEPS; ++s)
        if (s < n) issue(s, s);
    int slot = 0;
    for (int s = 0; s < n; ++s) {
        // step s has landed: all loads but those of the STEPS - 1 steps after it; near the end all of them
        // (s_waitcnt's gfx9 encoding: vmcnt in bits 0..3 and 14..15, the other counters at their maxima)
        constexpr int kAhead = (STEPS - 1) * 2 * (MB + NB);
        static_assert(kAhead < 64, "vmcnt has six bits");
        if (s + STEPS - 1 < n) __builtin_amdgcn_s_waitcnt(0x0F70 | (kAhead & 15) | ((kAhead >> 4) << 14));
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("" ::: "memory");
        const uint8_t *at = smem + w * (STEPS * kStepBytes) + slot * kStepBytes;
        v8i f[MB + NB];
#pragma unroll
        for (int b = 0; b < MB + NB; ++b) {
            const uint4 lo = *reinterpret_cast<const uint4 *>(at + b * kBlockBytes + frag_off[0]);
            const uint4 hi = *reinterpret_cast<const uint4 *>(at + b * kBlockBytes + frag_off[1]);
            f[b] = v8i{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);          // the fragments are in registers: the slot is free
        __builtin_amdgcn_sched_barrier(0);
        if (s + STEPS < n) issue(s + STEPS, slot);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[mb][nb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(f[mb], f[MB + nb], acc[mb][nb], AFMT, 0, 0, 0, 0, 0);
        slot = slot + 1 == STEPS ? 0 : slot + 1;
    }
    __syncthreads();                                 // every wave is done with its ring
    // register i of a lane: row (l >> 4) * 4 + i, column l & 15 of its block
    float *part = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                part[(w * (16 * MB) + mb * 16 + (l >> 4) * 4 + i) * kPitch + nb * 16 + (l & 15)] = acc[mb][nb][i];
    __syncthreads();

    const float s_a = p.sa ? *p.sa : 1.0f, s_b = p.sb ? *p.sb : 1.0f, s_b2 = kDual && p.sb2 ? *p.sb2 : 1.0f;
    const Dequant dq = inv_scale_product(s_a, s_b), dq2 = kDual ? inv_scale_product(s_a, s_b2) : dq;
    // a thread finishes two neighbouring columns
    for (int e = threadIdx.x; e < 16 * MB * (8 * NCOL); e += 64 * KW) {
        const int row = e / (8 * NCOL), c = e % (8 * NCOL) * 2;
        if (m0 + row >= p.M || n0 + c >= p.N) continue;
        float v[2][2];
#pragma unroll
        for (int h = 0; h < (kDual ? 2 : 1); ++h)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float *src = part + row * kPitch + h * (16 * NCOL) + c + k;
                float sum = src[0];
#pragma unroll
                for (int q = 1; q < KW; ++q) sum = __fadd_rn(sum, src[q * (16 * MB) * kPitch]);
                const Dequant &d = h == 0 ? dq : dq2;
                v[h][k] = __fmul_rn(sum, d.a);
                if (d.post != 1.0f) v[h][k] *= d.post;
            }
        const size_t at = (size_t)(m0 + row) * (size_t)p.N + (size_t)(n0 + c);
        if (kDual)
            *reinterpret_cast<uint16_t *>(reinterpret_cast<uint8_t *>(p.C) + at) =
                (uint16_t)satcast_pk2<kE4M3>(swiglu_f32(v[0][0], v[1][0]), swiglu_f32(v[0][1], v[1][1]));
        else if (p.c_f32) *reinterpret_cast<float2 *>(reinterpret_cast<float *>(p.C) + at) = make_float2(v[0][0], v[0][1]);
        else *reinterpret_cast<uint32_t *>(reinterpret_cast<uint16_t *>(p.C) + at) = pack_bf16x2(v[0][0], v[0][1]);
    }
}

template <int EPI, int AFMT, int MB, int NB, int KW, int STEPS>
__global__ void __launch_bounds__(64 * KW) gemm_skinny_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(1024))) uint8_t smem[skinny_smem(MB, NB, KW, STEPS)];
    gemm_skinny_block<EPI, AFMT, MB, NB, KW, STEPS>(p, blockIdx.x, smem);
}

// Gate/up of the inference form for a batch that ends a few rows after whole tiles: these run in the few-rows form, 16 * MB rows
// to a workgroup, in the same grid, in the slots that the tiles leave idle (their LDS fits beside a tile's).  Bound by the tiles,
// two on a compute unit; a row of 128-row tiles for 16 rows costs a half more (T = 272, d = 4096, f = 11008: 44 us in large tiles, the
// second row 1/16 full, 36 this way).  32 rows to a workgroup read the weights half as often as 16 (T = 288: 41 and 38; 320: 52 and 44).
template <int MB, int STEPS>
__global__ void __launch_bounds__(kThreads, 2) gemm_swiglu_q_rest_kernel(GemmParams p, GemmParams rest, int tile_blocks) {
    constexpr int kBytes = std::max(smem_bytes(2), skinny_smem(MB, 2, 4, STEPS));
    static_assert(2 * kBytes <= 163840, "two workgroups on a compute unit");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[kBytes];
    const int b = (int)blockIdx.x;
    if (b >= tile_blocks) {
        gemm_skinny_block<EPI_SWIGLU_Q, kE4M3, MB, 2, 4, STEPS>(rest, (unsigned)(b - tile_blocks), smem);
        return;
    }
    const int vb = set_of<2>(b) * 8 + (b & 7);
    if (vb < p.tiles_m * p.tiles_n) gemm_tile<2, EPI_SWIGLU_Q, kE4M3, 0, 0>(p, vb, quarter_of<2>(b), smem);
}

template <int EPI, int AFMT, int MB, int NB, int KW, int STEPS>
static void launch_form(const GemmParams &p, hipStream_t st) {
    constexpr int cols = 16 * (EPI == EPI_SWIGLU_Q ? NB / 2 : NB);
    const unsigned mblocks = (unsigned)((p.M + 16 * MB - 1) / (16 * MB)), nsets = (unsigned)((p.N + 8 * cols - 1) / (8 * cols));
    hipLaunchKernelGGL((gemm_skinny_kernel<EPI, AFMT, MB, NB, KW, STEPS>), dim3(mblocks * nsets * 8), dim3(64 * KW), 0, st, p);
}

// The forms: blocks of A and of B per workgroup, waves, steps of a wave's ring.  Of the plain store (the first six):
// larger ones fetch fewer bytes per product, smaller ones leave fewer compute units idle.  The last two are the SwiGLU form's.
constexpr int kStoreForms = 6;
static constexpr struct { int mb, nb, waves, steps; } kForms[] = {{1, 1, 4, 5}, {1, 2, 4, 3}, {2, 2, 4, 2}, {4, 2, 4, 3},
                                                                  {4, 4, 4, 2}, {6, 4, 4, 2}, {1, 2, 4, 3}, {4, 4, 2, 2}};

template <int EPI, int AFMT, int I>
static void launch_indexed(const GemmParams &p, hipStream_t st) {
    launch_form<EPI, AFMT, kForms[I].mb, kForms[I].nb, kForms[I].waves, kForms[I].steps>(p, st);
}

template <int AFMT>
static void launch_store(const GemmParams &p, int form, hipStream_t st) {
    switch (form) {
        case 0: launch_indexed<EPI_STORE, AFMT, 0>(p, st); break;
        case 1: launch_indexed<EPI_STORE, AFMT, 1>(p, st); break;
        case 2: launch_indexed<EPI_STORE, AFMT, 2>(p, st); break;
        case 3: launch_indexed<EPI_STORE, AFMT, 3>(p, st); break;
        case 4: launch_indexed<EPI_STORE, AFMT, 4>(p, st); break;
        default: launch_indexed<EPI_STORE, AFMT, 5>(p, st); break;
    }
}

// Microseconds of a form with B not in a cache: 4 to start and end, then each compute unit fetches 70 KB a microsecond
// for its share of the workgroups, and the whole chip 4.2 MB a microsecond from HBM; a quarter of the smaller of the two
// does not hide behind the larger.  (y of the inference form, N = 4096, K = 11008, estimated / measured: T = 16 form
// {1,1} 16 / 14, T = 32 {1,2} 17 / 16, T = 64 {2,2} 17 / 19, T = 128 {4,2} 22 / 24, T = 208 {4,4} 27 / 26, T = 272
// {6,4} 32 / 33; the 128 x 128 tile with its longer ring takes 42 to 57 for all of them.)  More workgroups than compute
// units pay the 4 each round, and a third more per byte (1040 x 2736 x 4096, two rounds of {6,4}: 35 / 39; tile: 22).
// Rounds are counted on the XCD that has most: all row blocks of one column block go to the same, so 128 columns in blocks
// of 64 are the work of two XCDs (6400 x 128 x 256: 17.6 us in {4,4}, 7.2 in 128 x 128 tiles).
static double form_time(const GemmArgs &a, int form) {
    const int64_t m = 16 * kForms[form].mb, n = 16 * kForms[form].nb;
    const int64_t groups = ((a.M + m - 1) / m) * (((a.N + n - 1) / n + 7) / 8), rounds = (groups + kComputeUnits / 8 - 1) / (kComputeUnits / 8);
    const double fetch = (double)((m + n) * a.K) / 70e3, hbm = (double)(a.N * a.K) / 4.2e6;
    const double busy = rounds == 1 ? fetch : (double)rounds * (1.35 * fetch + 4.0) - 4.0;
    return 4.0 + std::max(busy, hbm) + 0.25 * std::min(busy, hbm);
}

// The SwiGLU form: up to 128 rows (gate/up of the inference form against the 128 x 128 tile, us, d = 4096, f = 11008: T = 16
// 22 against 36, T = 64 27 against 40, T = 128 44 against 48, T = 208 53 against 43; d = 2048, f = 5504: T = 128 15 against
// 18, T = 272 24 against 22), and so many workgroups that each compute unit runs at most 4.5 of them one after the other
// (against large tiles: d = 4864, f = 17760, 140 on an XCD, T = 96 49 and 52; d = 2048, f = 28672, 224, 38 and 33;
// d = 7680, f = 24592, 194, 126 and 99).  Rows that do not start on 128-byte lines cost both its waves two lines per piece:
// less of them by what a compute unit fetches (d = 4656, f = 11680, T = 80: 70 and 81; d = 7120, f = 19216, T = 64: 119 and
// 101; d = 7760, f = 24752, T = 96: 170 and 116).
static bool swiglu_form_ok(const GemmArgs &a) {
    if (a.M <= 16) return true;
    const int64_t rows = 16 * kForms[kStoreForms + 1].mb, cols = 8 * kForms[kStoreForms + 1].nb;
    const int64_t on_xcd = ((a.M + rows - 1) / rows) * (((a.N + cols - 1) / cols + 7) / 8);
    return a.M <= 128 && on_xcd <= 9 * kComputeUnits / 16 && (a.K % 128 == 0 || on_xcd * a.K <= 450000);
}

// K-contiguous FP8 operands, the plain store without a per-column factor or the inference form's SwiGLU.
double gemm_skinny_time(const GemmArgs &a, int *form) {
    const double never = 1e30;
    *form = 0;
    if (a.layout != 0 || a.part != 0 || a.a_fmt == kBF16 || a.col_scale) return never;
    if (a.epilogue == EPI_SWIGLU_Q) {
        *form = a.M <= 16 ? kStoreForms : kStoreForms + 1;
        return swiglu_form_ok(a) ? 0.0 : never;
    }
    if (a.epilogue != EPI_STORE) return never;
    double best = form_time(a, 0);
    for (int i = 1; i < kStoreForms; ++i) {
        const double t = form_time(a, i);
        if (t < best) { best = t; *form = i; }
    }
    return best;
}

void launch_gemm_skinny(const GemmArgs &a, int form, hipStream_t st) {
    const GemmParams p = make_gemm_params(a);
    if (form == kStoreForms) launch_indexed<EPI_SWIGLU_Q, kE4M3, kStoreForms>(p, st);
    else if (form > kStoreForms) launch_indexed<EPI_SWIGLU_Q, kE4M3, kStoreForms + 1>(p, st);
    else if (a.a_fmt == kE4M3) launch_store<kE4M3>(p, form, st);
    else launch_store<kE5M2>(p, form, st);
}

void launch_gemm_rest(const GemmArgs &a, int rows, hipStream_t st) {
    GemmArgs main = a, rest = a;
    main.M = a.M - rows;
    rest.M = rows;
    rest.A = a.A + (size_t)main.M * (size_t)a.K;
    rest.C = static_cast<uint8_t *>(a.C) + (size_t)main.M * (size_t)a.N;
    const GemmParams p = make_gemm_params(main), q = make_gemm_params(rest);
    // (column blocks in sets of 8, one to an XCD, the row blocks of one after the other)
    const int block = few_last_block(rows);
    const unsigned blocks = (unsigned)sets_of(p) * set_workgroups(2), more = (unsigned)((a.N + 127) / 128 * ((rows + block - 1) / block)) * 8u;
    if (block == 16) hipLaunchKernelGGL((gemm_swiglu_q_rest_kernel<1, 3>), dim3(blocks + more), dim3(kThreads), 0, st, p, q, (int)blocks);
    else hipLaunchKernelGGL((gemm_swiglu_q_rest_kernel<2, 2>), dim3(blocks + more), dim3(kThreads), 0, st, p, q, (int)blocks);
}

void gemm_skinny_extent(const GemmArgs &a, int form, int *rows, int *cols, int *steps) {
    *rows = 16 * kForms[form].mb;
    *cols = 16 * kForms[form].nb / (a.epilogue == EPI_SWIGLU_Q ? 2 : 1);
    *steps = kForms[form].steps;
}

}  // namespace ssg
