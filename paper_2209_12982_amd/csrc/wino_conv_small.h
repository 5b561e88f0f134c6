// The whole convolution in one launch for small layers, int8 operands, 32-bit
// epilogue: wino_conv_small.  Included by wino_kernels.hip inside its anonymous
// namespace.
//
// On a small layer the input transform and the tap GEMM each last little longer
// than a launch and two memory round trips.  Here a workgroup of 16 CB channels x
// 16 tiles transforms its own tiles (B^T d B, tap-wise requantization) into LDS,
// 64 input channels at a time, and runs wino_tap_gemm_small's row-of-taps waves
// on them: wave a takes row a of the taps, Uq fragments straight from memory, Vq
// fragments from LDS, then the row pass to LDS and the column pass, requantize,
// store.  The next chunk's pixels and weights are loaded while this one computes.
// The transform is repeated by every block of output channels, which pays as
// long as the blocks run at once (the rule at launch).
template <int M, int CB>
struct CsCfg {
    static constexpr int N = M + 2, NT = N * N, CO = 16 * CB, THREADS = 64 * N;
    static constexpr int PITCH = CO + 4;
    static constexpr int V_BYTES = NT * 16 * 64;           // one chunk of 16 tiles
    static constexpr int Z_BYTES = N * M * 16 * PITCH * 4;
    static constexpr int LDS = V_BYTES + Z_BYTES;
    static_assert(LDS <= 160 * 1024, "LDS");
};

struct CsArgs {
    K2Args k;                                              // as for the tap GEMM
    int cin, x_bytes, q_sat;
    uint32_t rnd2[kTaps];
};

// Raw words of the N x N window of four channels ci .. ci + 3 of a tile.  NHWC: one
// word per pixel; NCHW: NW words per channel and window row, at columns x0 and
// (N = 6) x0 + 2.
template <int M, int LAYOUT>
struct CsWin {
    static constexpr int N = M + 2, NW = N == 4 ? 1 : 2;
    static constexpr int WORDS = LAYOUT == WINO_NHWC ? N * N : 4 * N * NW;
};

template <int M, int LAYOUT>
using CsRaw = uint32_t[CsWin<M, LAYOUT>::WORDS];

// Issue the loads.  Words that stick out of a pixel's channels (NHWC) or of the
// image row (NCHW) are read from inside and shifted by cs_finish; words wholly
// outside read as zero.
template <int M, int LAYOUT>
__device__ __forceinline__ void cs_load(CsRaw<M, LAYOUT>& raw, __amdgpu_buffer_rsrc_t rs, const CsArgs& g,
                                        bool ok, int img, int ty, int tx, int ci) {
    constexpr int N = M + 2, NW = CsWin<M, LAYOUT>::NW;
    constexpr int kOut = 0x7ffffff0;                       // past the tensor (checked on the host)
    const int h = g.k.h, w = g.k.w, y0 = M * ty - 1, x0 = M * tx - 1;
    if constexpr (LAYOUT == WINO_NHWC) {
        const int base = ((img * h + y0) * w + x0) * g.cin + min(ci, g.cin - 4);   // Cin >= 4
        ok = ok && ci < g.cin;
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int c = 0; c < N; ++c) {
                const bool in = ok && y0 + r >= 0 && y0 + r < h && x0 + c >= 0 && x0 + c < w;
                raw[N * r + c] = __builtin_amdgcn_raw_buffer_load_b32(rs, in ? base + (r * w + c) * g.cin : kOut, 0, 0);
            }
    } else {
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int c4 = x0 + 2 * k, col = max(0, min(c4, w - 4));               // W >= 4
#pragma unroll
            for (int r = 0; r < N; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = ok && ci + e < g.cin && y0 + r >= 0 && y0 + r < h && c4 < w;
                    raw[(r * 4 + e) * NW + k] = __builtin_amdgcn_raw_buffer_load_b32(
                        rs, in ? ((img * g.cin + ci + e) * h + y0 + r) * w + col : kOut, 0, 0);
                }
        }
    }
}

// wv[r][c] = the four channels of window pixel (r, c), one byte each
template <int M, int LAYOUT, int N = Wino<M>::N>
__device__ __forceinline__ void cs_finish(uint32_t (&wv)[N][N], const CsRaw<M, LAYOUT>& raw,
                                          const CsArgs& g, int tx, int ci) {
    constexpr int NW = CsWin<M, LAYOUT>::NW;
    if constexpr (LAYOUT == WINO_NHWC) {
        const int sh = 8 * (ci - min(ci, g.cin - 4)) & 31;  // 0 for whole words; past Cin the words are zero
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int c = 0; c < N; ++c) wv[r][c] = raw[N * r + c] >> sh;
    } else {
        const int w = g.k.w, x0 = M * tx - 1;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int c4 = x0 + 2 * k, col = max(0, min(c4, w - 4));
            const int left = 8 * max(col - c4, 0), right = 8 * max(c4 - col, 0) & 31;
#pragma unroll
            for (int r = 0; r < N; ++r) {
                uint32_t v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = raw[(r * 4 + e) * NW + k] >> right << left;
                const uint32_t ab_lo = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u);
                const uint32_t ab_hi = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
                const uint32_t cd_lo = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u);
                const uint32_t cd_hi = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
                const uint32_t quad[4] = {__builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u),
                                          __builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u),
                                          __builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u),
                                          __builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u)};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k == 0 || j >= 2) wv[r][2 * k + j] = quad[j];
            }
        }
    }
}

template <int M, int CB, int LAYOUT, bool SAT>
__global__ __launch_bounds__(64 * (M + 2), 2) void wino_conv_small(const int8_t* __restrict__ x,
                                                                   const int8_t* __restrict__ uq,
                                                                   const int32_t* __restrict__ bias,
                                                                   int8_t* __restrict__ y, CsArgs ga) {
    typedef CsCfg<M, CB> C;
    constexpr int N = C::N, NT = C::NT, TL = 16;
    constexpr uint32_t kAdd2 = 0x00800080u;                // see k1_store, Q = 8
    const K2Args& g = ga.k;
    __shared__ __attribute__((aligned(1024))) uint8_t vs[C::V_BYTES];     // [tap][tile][64], 16-byte slots swizzled
    __shared__ __attribute__((aligned(16))) int zs[N][M][TL][C::PITCH];
    const int lane = threadIdx.x & 63;
    const int a = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // this wave's row of taps
    const int lr = lane & 15, lk = lane >> 4;
    const int nkc = g.cin_pad / kKStep;
    const uint32_t lbid = (uint32_t)xcd_remap(blockIdx.x, g.nblocks);
    const uint32_t btl = fast_div(lbid, g.dgco), bco = lbid - btl * g.dgco.d;
    const int co_blk = (int)bco * C::CO;
    const long long tl_blk = (long long)btl * TL;

    // transform side: threads 0-255 take tile t / 16, channels 4 (t % 16) .. + 3
    const int q = threadIdx.x & 15, vt = (threadIdx.x >> 4) & 15;
    const bool xform = threadIdx.x < 256;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, ga.x_bytes, 0x00020000);
    int img = 0, ty = 0, tx = 0;
    const bool tile_ok = xform && tl_blk + vt < g.ntiles;
    if (tile_ok) tile_coords(tl_blk + vt, g, img, ty, tx);
    CsRaw<M, LAYOUT> raw;
    if (xform) cs_load<M, LAYOUT>(raw, rs, ga, tile_ok, img, ty, tx, 4 * q);
    uint8_t* const vdst = vs + vt * 64 + 16 * lds_slot(vt, q >> 2) + 4 * (q & 3);

    // compute side
    const uint32_t lane_off = (uint32_t)(lr * 64 + lk * 16);
    const long long su = (long long)g.cout_pad * g.cin_pad, ku = (long long)g.cout_pad * kKStep;
    const int8_t* ub = uq + (long long)co_blk * kKStep + N * a * su;
    const uint8_t* const vsrc = vs + N * a * TL * 64 + lr * 64 + 16 * lds_slot(lr, lk);
    v4i fa[N][CB], m[N][CB];
    auto load_u = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CB; ++c) fa[b][c] = *(const v4i*)(ub + b * su + 1024 * c + lane_off);
    };
#pragma unroll
    for (int b = 0; b < N; ++b) load_u(b);
    const int rnd = g.out_shift > 0 ? 1 << (g.out_shift - 1) : 0;
    v4i bias_rnd[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) bias_rnd[c] = *(const v4i*)(bias + co_blk + 16 * c + 4 * lk) + rnd;
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < CB; ++c) m[b][c] = (v4i){0, 0, 0, 0};

    for (int kc = 0; kc < nkc; ++kc) {
        if (xform) {
            uint32_t wv[N][N];
            cs_finish<M, LAYOUT>(wv, raw, ga, tx, 64 * kc + 4 * q);
            if (kc + 1 < nkc) cs_load<M, LAYOUT>(raw, rs, ga, tile_ok, img, ty, tx, 64 * (kc + 1) + 4 * q);
            v2s ev[N][N], od[N][N];
            input_tile_transform<M>(wv, ev, od);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint32_t v =
                    SAT ? requant_pack_sat(ev[t / N][t % N], od[t / N][t % N], (1u << (8 - g.tab.eb[t])) * 0x10001u, kAdd2)
                        : requant_pack(ev[t / N][t % N], od[t / N][t % N], g.tab.eb[t], ga.rnd2[t]);
                *(uint32_t*)(vdst + t * TL * 64) = v;
            }
        }
        __syncthreads();                                   // the chunk's Vq is in LDS
        ub += ku;
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const v4i fb = *(const v4i*)(vsrc + b * TL * 64);
#pragma unroll
            for (int c = 0; c < CB; ++c) m[b][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[b][c], fb, m[b][c], 0, 0, 0);
            if (kc + 1 < nkc) load_u(b);
        }
        __syncthreads();                                   // and read by every wave
    }

    // row pass: lane holds channels 16 c + 4 lk + r of tile lr
    int sh[N];
#pragma unroll
    for (int b = 0; b < N; ++b) sh[b] = g.tab.sh[N * a + b];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        v4i z[M];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int mv[N], zr[M];
#pragma unroll
            for (int b = 0; b < N; ++b) mv[b] = m[b][c][r] << sh[b];
            if (a == 1) mv[1] += bias_rnd[c][r];
            Wino<M>::at(mv, zr);
#pragma unroll
            for (int j = 0; j < M; ++j) z[j][r] = zr[j];
        }
#pragma unroll
        for (int j = 0; j < M; ++j) *(v4i*)&zs[a][j][lr][16 * c + 4 * lk] = z[j];
    }
    __syncthreads();
    uint32_t zmax = 0;
    small_column_pass<M, C::CO, TL, C::THREADS, LAYOUT, 0>(zs, g, y, co_blk, tl_blk, zmax);
}
