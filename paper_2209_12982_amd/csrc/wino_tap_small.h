// Tap GEMM + output transform for layers with few blocks, int8 operands,
// 32-bit epilogue: wino_tap_gemm_small, F(4x4,3x3) and F(2x2,3x3).  Included by
// wino_kernels.hip inside its anonymous namespace.
//
// Such a layer is bound by latency, not by a rate: with 64 x 32 blocks most
// compute units idle (8x32x32, 128->128: 32 blocks on 256) and a block walks a
// serial chain of ring stages, a barrier each, and an epilogue in which every
// lane folds four whole channels.  Here
//   * a block is 16 CB channels x 16 TB tiles, 16 x 16 to 32 x 32, so that the
//     layer has about one per compute unit or more;
//   * wave a of the M + 2 waves owns row a of the taps and accumulates its
//     M + 2 tap GEMMs over all input channels, so the taps run side by side;
//   * operand fragments go from memory straight to registers: 16 rows x 64 bytes
//     of the k-blocked operands are one contiguous 1-KB load, already in the
//     MFMA's layout.  No LDS ring and no barrier in the loop; a whole 64-channel
//     chunk of the row's taps is in flight per wave;
//   * wave a then folds its row, z_a = (M'[a, :]) A (M' = M 2^sh), into LDS, and
//     all waves apply the column pass Y = A^T z, requantize and store.
// Every operand byte is read by 16 CB or 16 TB columns only, so large F4 layers
// run the LDS-staged row-streamed kernel, and F2 layers the staged 64 x 32 blocks
// where these need no more rounds or Vq lies beyond the caches (the rules at
// launch).
// Measured against the 64 x 32 blocks it replaces (kernel time, us): F4 8x32x32
// 128->128 16.2 -> 5.6, 256->512 22.5 -> 13.6, 2x75x75 256->256 26.0 -> 16.2; F2
// 8x56x56 64->64 6.1 -> 5.9, 8x14x14 256->256 10.0 -> 6.4, 8x112x112 64->64 19.8
// -> 12.4, 256x256 128->128 26.0 -> 20.8.  What is left at the small sizes is the
// launch and two memory round trips (2.5 K clk each).
template <int M, int CB, int TB>
struct TsCfg {
    static constexpr int N = M + 2, CO = 16 * CB, TL = 16 * TB, THREADS = 64 * N;
    static constexpr int PITCH = CO + 4;                  // int32 per (row, column, tile); the pad spreads banks
    static constexpr int LDS = N * M * TL * PITCH * 4;
    static_assert(LDS <= 160 * 1024, "LDS");
};

// The column pass of a block's row-pass results zs (bias and rounding constant
// included): Y = A^T z, then requantize and store (MODE 0), or the maximum of |Y|
// over the in-image outputs into zmax (MODE 1).
template <int M, int CO, int TL, int THREADS, int LAYOUT, int MODE>
__device__ __forceinline__ void small_column_pass(const int (&zs)[M + 2][M][TL][CO + 4], const K2Args& g,
                                                  int8_t* __restrict__ y, int co_blk, long long tl_blk, uint32_t& zmax) {
    constexpr int N = M + 2;
    if constexpr (LAYOUT == WINO_NHWC) {
        // column pass, one item per (tile, column j, four channels): M pixels of
        // four channels each
        const bool word = (g.cout & 3) == 0 && ((uintptr_t)y & 3) == 0;
        constexpr int QC = CO / 4;
        for (int id = threadIdx.x; id < TL * M * QC; id += THREADS) {
            const int q = id % QC, j = id / QC % M, tl = id / (QC * M);
            const long long tile = tl_blk + tl;
            const int co = co_blk + 4 * q;
            if (tile >= g.ntiles || co >= g.cout) continue;
            v4i zv[N];
#pragma unroll
            for (int b = 0; b < N; ++b) zv[b] = *(const v4i*)&zs[b][j][tl][4 * q];
            int o[4][M];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int col[N];
#pragma unroll
                for (int b = 0; b < N; ++b) col[b] = zv[b][r];
                Wino<M>::at(col, o[r]);
            }
            int img, ty, tx;
            tile_coords(tile, g, img, ty, tx);
            const int xx = M * tx + j;
            if (xx >= g.w) continue;
            int8_t* p = y + (((long long)img * g.h + M * ty) * g.w + xx) * g.cout + co;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if (M * ty + i >= g.h) break;
                if constexpr (MODE == 1) {                 // channels past Cout hold zeros
#pragma unroll
                    for (int r = 0; r < 4; ++r) zmax = max(zmax, (uint32_t)abs(o[r][i]));
                    continue;
                }
                uint32_t w = join2(requant2(o[0][i], o[1][i], g.out_shift), requant2(o[2][i], o[3][i], g.out_shift));
                if (g.relu) w = relu4(w);
                if (word) {
                    *(uint32_t*)p = w;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (co + r < g.cout) p[r] = (int8_t)(w >> (8 * r));
                }
                p += (long long)g.w * g.cout;
            }
        }
    } else {
        // one item per (channel, tile), tiles fastest: M rows of M pixels
        const bool word = g.w % M == 0 && ((uintptr_t)y & (M - 1)) == 0;
        for (int id = threadIdx.x; id < TL * CO; id += THREADS) {
            const int tl = id % TL, ch = id / TL;
            const long long tile = tl_blk + tl;
            const int co = co_blk + ch;
            if (tile >= g.ntiles || co >= g.cout) continue;
            int o[M][M];                                   // [column][row]
#pragma unroll
            for (int j = 0; j < M; ++j) {
                int col[N];
#pragma unroll
                for (int b = 0; b < N; ++b) col[b] = zs[b][j][tl][ch];
                Wino<M>::at(col, o[j]);
            }
            int img, ty, tx;
            tile_coords(tile, g, img, ty, tx);
            int8_t* p = y + (((long long)img * g.cout + co) * g.h + M * ty) * g.w + M * tx;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if (M * ty + i >= g.h) break;
                uint32_t w = requant2(o[0][i], o[1][i], g.out_shift);
                if constexpr (M == 4) w = join2(w, requant2(o[2][i], o[3][i], g.out_shift));
                if (g.relu) w = relu4(w);
                if (word) {
                    if constexpr (M == 4) *(uint32_t*)p = w;
                    else *(uint16_t*)p = (uint16_t)w;
                } else {
#pragma unroll
                    for (int j = 0; j < M; ++j)
                        if (M * tx + j < g.w) p[j] = (int8_t)(w >> (8 * j));
                }
                p += g.w;
            }
        }
    }
}

// MODE 0: store y.  MODE 1: max |Y + bias| into *aux (calibration).
template <int M, int CB, int TB, int LAYOUT, int MODE>
__global__ __launch_bounds__(64 * (M + 2), 2) void wino_tap_gemm_small(const int8_t* __restrict__ uq,
                                                                       const int8_t* __restrict__ vq,
                                                                       const int32_t* __restrict__ bias,
                                                                       int8_t* __restrict__ y,
                                                                       void* __restrict__ aux, K2Args g) {
    typedef TsCfg<M, CB, TB> C;
    constexpr int N = C::N;
    __shared__ __attribute__((aligned(16))) int zs[N][M][C::TL][C::PITCH];
    const int lane = threadIdx.x & 63;
    const int a = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // this wave's row of taps
    const int lr = lane & 15, lk = lane >> 4;
    const int nkc = g.cin_pad / kKStep;
    const uint32_t lbid = (uint32_t)xcd_remap(blockIdx.x, g.nblocks);
    const uint32_t grp = min(fast_div(lbid, g.dgrp), (uint32_t)g.nfull);
    const uint32_t rem = lbid - grp * g.dgrp.d;
    const bool full = grp < (uint32_t)g.nfull;
    const uint32_t btl = fast_div(rem, full ? g.dgco : g.drest);
    const uint32_t bco = grp * g.gco + (rem - btl * (full ? g.dgco.d : g.drest.d));
    const int co_blk = (int)bco * C::CO;
    const long long tl_blk = (long long)btl * C::TL;

    const uint32_t lane_off = (uint32_t)(lr * 64 + lk * 16);
    const long long su = (long long)g.cout_pad * g.cin_pad, sv = g.t_pad * g.cin_pad;   // tap strides
    const long long ku = (long long)g.cout_pad * kKStep, kv = g.t_pad * kKStep;           // k-chunk strides
    const int8_t* ub = uq + (long long)co_blk * kKStep + N * a * su;
    const int8_t* vb = vq + tl_blk * kKStep + N * a * sv;
    v4i fa[N][CB], fb[N][TB], m[N][CB][TB];
    auto load = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CB; ++c) fa[b][c] = *(const v4i*)(ub + b * su + 1024 * c + lane_off);
#pragma unroll
        for (int t = 0; t < TB; ++t) fb[b][t] = *(const v4i*)(vb + b * sv + 1024 * t + lane_off);
    };
#pragma unroll
    for (int b = 0; b < N; ++b) load(b);
    // bias plus rounding constant, injected through tap (1,1): its row and
    // column of A^T are all ones, so it reaches every output of the tile once
    const int rnd = MODE == 0 && g.out_shift > 0 ? 1 << (g.out_shift - 1) : 0;
    v4i bias_rnd[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) bias_rnd[c] = *(const v4i*)(bias + co_blk + 16 * c + 4 * lk) + rnd;
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int t = 0; t < TB; ++t) m[b][c][t] = (v4i){0, 0, 0, 0};
    for (int kc = 1; kc < nkc; ++kc) {
        ub += ku;
        vb += kv;
#pragma unroll
        for (int b = 0; b < N; ++b) {
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int t = 0; t < TB; ++t)
                    m[b][c][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[b][c], fb[b][t], m[b][c][t], 0, 0, 0);
            load(b);                                       // the next chunk's
        }
    }
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int t = 0; t < TB; ++t)
                m[b][c][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[b][c], fb[b][t], m[b][c][t], 0, 0, 0);

    // row pass: lane holds channels 16 c + 4 lk + r of tile 16 t + lr
    int sh[N];
#pragma unroll
    for (int b = 0; b < N; ++b) sh[b] = g.tab.sh[N * a + b];
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            v4i z[M];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int mv[N], zr[M];
#pragma unroll
                for (int b = 0; b < N; ++b) mv[b] = m[b][c][t][r] << sh[b];
                if (a == 1) mv[1] += bias_rnd[c][r];
                Wino<M>::at(mv, zr);
#pragma unroll
                for (int j = 0; j < M; ++j) z[j][r] = zr[j];
            }
#pragma unroll
            for (int j = 0; j < M; ++j) *(v4i*)&zs[a][j][16 * t + lr][16 * c + 4 * lk] = z[j];
        }
    __syncthreads();

    uint32_t zmax = 0;
    small_column_pass<M, C::CO, C::TL, C::THREADS, LAYOUT, MODE>(zs, g, y, co_blk, tl_blk, zmax);
    if constexpr (MODE == 1) {
        __syncthreads();                                   // zs is read no more
        block_max<C::THREADS / 64>(zmax, (uint32_t*)zs, (unsigned long long*)aux);
    }
}
