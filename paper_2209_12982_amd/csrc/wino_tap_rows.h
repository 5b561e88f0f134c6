// Tap GEMM + output transform for F(4x4,3x3), int8 operands, 32-bit
// epilogue: the row-streamed kernel wino_tap_gemm_rows.  Included by
// wino_kernels.hip inside its anonymous namespace.
//
// Y = A^T M' A is linear in the taps, and its row pass only mixes the six
// taps of one row a of the 6x6 tile: with z_a = (M'[a, :]) A, Y = sum_a
// A^T[:, a] z_a.  So the taps stream row by row: the six M_t of row a
// accumulate over all input channels, fold into z_a, and their accumulators
// serve the next row.
//
// Order of the rows.  Columns 1 and 2 of A^T (and 3 and 4) differ only in the
// signs of the odd output rows, so rows 1 and 2 enter Y as p = z1 + z2 (even
// output rows) and m = z1 - z2 (odd ones), rows 3 and 4 as q = z3 + z4 and
// r = z3 - z4:
//   Y0 = z0 + p + q, Y1 = m + 2 r, Y2 = p + 4 q, Y3 = z5 + m + 8 r.
// Taken as 1, 2, 3, 4, 0, 5, a (tile, channel) pair keeps p and m (8 values),
// then z3 beside them; after row 4 the output rows 1 and 2 are final and are
// requantized to packed bytes at once, p + q and m + 8 r remain, and rows 0
// and 5 finish output rows 0 and 3.  That is 12 int32 per pair at the most
// next to the row's six accumulators, where adding every z_a into a 4x4 Y
// needs 16, and 16 additions per row pair instead of 32.
//
// Integer arithmetic is exact: the 32-bit epilogue is only selected when the
// plan's bound on the sum of the terms' magnitudes, which bounds every
// partial sum above, is below 2^31.
//
// What bounds it, 4x256->256 160x160, a 64x64 block of 24 stages: the operand
// copies alone take 27 K clk (43 B/clk per CU), everything but the copies 28 K, the
// loop with both 32 K, the epilogue 9 K.  Kernel time there 39.4 us (768 TOP/s;
// 48.6 in a 16-wave form that issued a stage's copies in a row and folded each row
// after its last stage), 16.9 us at 1x128->128 256x512 (19.9), 20.0 us at 1x64->64
// 568x568 (26.8).
constexpr int RW_CB = 2;                                  // 16-channel blocks per wave
constexpr int RW_CO = 64;
constexpr int RW_V = 4 * RW_CB;                           // pairs per lane
// Block of 64 channels x TL tiles, a wave 32 x 16 of it; ring of NBUF stages of
// G taps of a row x 64 input channels.
template <int TL_, int G_, int NBUF_>
struct RwCfg {
    static constexpr int TL = TL_, G = G_, NBUF = NBUF_, WAVES = 2 * TL / 16, THREADS = 64 * WAVES;
    static constexpr int SPR = 6 / G;                     // stages per row of taps and k-chunk
    static constexpr int SLICE = (RW_CO + TL) * kKStep;   // one tap, one k-chunk
    static constexpr int STAGE = G * SLICE;
    static constexpr int LPW = TL == 64 ? G : 5;          // copies per wave per stage
    static_assert(TL == 64 || (TL == 32 && G == 3), "copy maps");
    static_assert(6 % G == 0 && RW_CB * 16 * 2 == RW_CO, "stages split a row, waves the block");
    static_assert(NBUF * STAGE + 4 * RW_CO <= (TL == 64 ? 160 : 80) * 1024, "one or two workgroups per CU");
    static_assert((NBUF - 1) * LPW <= 63, "vmcnt range");
    static_assert(kTilePad % TL == 0 && kCoutPad % RW_CO == 0, "blocks tile the padded sizes");
};

enum { RW_COPY, RW_ASK };

// global -> LDS copy of 16 bytes per lane as lds_copy16, with the address as
// a wave-uniform 64-bit base and a 32-bit lane offset.  No memory clobber: the
// ring's barriers order it against the LDS reads of its buffer, and reads of
// the other buffers may move across it.
__device__ __forceinline__ void lds_copy16_s(const void* base, uint32_t lane_off,
                                             __attribute__((address_space(3))) void* dst) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "{m0}"(m0));
}

// two int32 (rounding constant included) -> clamp(v >> s, -128, 127), packed
// in the low half; two such halves -> one word
__device__ __forceinline__ uint32_t requant2(int a, int b, int s) {
    return __builtin_amdgcn_ashr_pk_i8_i32(a, b, s);
}
__device__ __forceinline__ uint32_t join2(uint32_t lo, uint32_t hi) {
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
// max(byte, 0) of the four signed bytes of w
__device__ __forceinline__ uint32_t relu4(uint32_t w) {
    const uint32_t t = w & 0x80808080u;
    return w & ~(t | (t - (t >> 7)));
}

// lds_copy16_s for lanes 0-31 only (512 bytes)
__device__ __forceinline__ void lds_copy16_half(const void* base, uint32_t lane_off,
                                                __attribute__((address_space(3))) void* dst) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
    asm volatile("s_mov_b32 exec_hi, 0\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b32 exec_hi, -1" ::"v"(lane_off),
                 "s"(base), "{m0}"(m0));
}

// maximum of zmax over the workgroup's W waves into *out, one atomic
template <int W>
__device__ __forceinline__ void block_max(uint32_t zmax, uint32_t* lds, unsigned long long* out) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) zmax = max(zmax, (uint32_t)__shfl_xor((int)zmax, off, 64));
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = zmax;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < W; ++w) zmax = max(zmax, lds[w]);
        atomicMax(out, (unsigned long long)zmax);
    }
}

// ONE: a single 64-channel chunk (Cin <= 64).
// MODE 0: store y.  MODE 1: max |Y + bias| into *aux (calibration).
template <class C, int LAYOUT, bool ONE, int MODE>
__global__ __launch_bounds__(C::THREADS, 2) void wino_tap_gemm_rows(
    const int8_t* __restrict__ uq, const int8_t* __restrict__ vq, const int32_t* __restrict__ bias,
    int8_t* __restrict__ y, void* __restrict__ aux, K2Args g) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[C::NBUF * C::STAGE];
    __shared__ __attribute__((aligned(16))) int bias_blk[RW_CO];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cw = wave & 1, tw = wave >> 1;
    const int lr = lane & 15, lk = lane >> 4;
    const int nkc = ONE ? 1 : g.cin_pad / kKStep;
    const int nstage = 6 * C::SPR * nkc;
    const int lbid = xcd_remap(blockIdx.x, g.nblocks);
    const int bco = lbid % g.nbco, btl = lbid / g.nbco;
    const int co_blk = bco * RW_CO;
    const long long tl_blk = (long long)btl * C::TL;
    // the block's bias into LDS as the first copy of the ring, which the wait
    // for stage 0 covers (vmcnt counts in order): loaded through a register, it
    // would hold the ring's start up for a memory round trip
    if (wave == 0) {
        const uint32_t m0 = __builtin_amdgcn_readfirstlane(
            (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)bias_blk);
        asm volatile("s_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(4 * lane), "s"(bias + co_blk), "{m0}"(m0)
                     : "memory");
    }

    // copy side (k-blocked operands Uq[36][cin_pad/64][cout_pad][64],
    // Vq[36][cin_pad/64][t_pad][64]).  A slice is 64 Uq and TL Vq rows.
    // TL = 64: wave w copies row group w (16 rows; 0-3: Uq, 4-7: Vq) of each of a
    // stage's slices (source u).  TL = 32 (three slices): wave w copies Uq rows
    // 16 w .. 16 w + 15 of each (source u), and of Vq (source v) rows 16 (w % 2) ..
    // of slice w / 2 and rows 8 w .. 8 w + 7 of slice 2.
    const int rr = lane >> 2;
    const uint32_t lane_off = (uint32_t)(rr * 64 + 16 * lds_slot(rr, lane & 3));
    const long long su = (long long)g.cout_pad * g.cin_pad, sv = g.t_pad * g.cin_pad;   // tap strides
    const long long ku = (long long)g.cout_pad * kKStep, kv = g.t_pad * kKStep;           // k-chunk strides
    const bool u_is_v = C::TL == 64 && wave >= 4;
    const long long ts = u_is_v ? sv : su, ks = u_is_v ? kv : ku;
    const int8_t* const u0 = u_is_v ? vq + (tl_blk + 16 * (wave - 4)) * kKStep
                                    : uq + (long long)(co_blk + 16 * wave) * kKStep;
    const int8_t* const v0 = vq + tl_blk * kKStep;
    const long long v_full = (wave >> 1) * sv + 1024 * (wave & 1), v_half = 2 * sv + 512 * wave;
    const int dst_u = 1024 * wave;
    const int dst_full = (wave >> 1) * C::SLICE + RW_CO * kKStep + 1024 * (wave & 1);
    const int dst_half = 2 * C::SLICE + RW_CO * kKStep + 512 * wave;
    constexpr uint32_t kRowOrder = 0x504321u;             // rows of taps in stream order, 4 bits each
    const int8_t* next_u = u0 + 6 * ts;
    const int8_t* next_v = v0 + 6 * sv;
    uint32_t rows_left = kRowOrder >> 4;
    int next_kc = 0, wr_off = 0;
    // part i (0 .. G - 1) of the next stage's copies
    auto issue_part = [&](int i) __attribute__((always_inline)) {
        uint8_t* const d = lds + wr_off;
        lds_copy16_s(next_u + i * ts, lane_off, (__attribute__((address_space(3))) void*)(d + i * C::SLICE + dst_u));
        if (C::TL == 32 && i == 0)
            lds_copy16_s(next_v + v_full, lane_off, (__attribute__((address_space(3))) void*)(d + dst_full));
        if (C::TL == 32 && i == 1)
            lds_copy16_half(next_v + v_half, lane_off, (__attribute__((address_space(3))) void*)(d + dst_half));
    };
    // step the copy side from stage j of a row of taps and k-chunk to the next
    auto issue_end = [&](int j) __attribute__((always_inline)) {
        if (j < C::SPR - 1) {
            next_u += C::G * ts;
            if (C::TL == 32) next_v += C::G * sv;
        } else if (++next_kc == nkc) {
            next_kc = 0;
            const int a = rows_left & 15;
            next_u = u0 + (long long)(6 * a) * ts;
            if (C::TL == 32) next_v = v0 + (long long)(6 * a) * sv;
            rows_left >>= 4;
        } else {
            next_u += ks - C::G * (C::SPR - 1) * ts;
            if (C::TL == 32) next_v += kv - C::G * (C::SPR - 1) * sv;
        }
        wr_off = wr_off == (C::NBUF - 1) * C::STAGE ? 0 : wr_off + C::STAGE;
    };

    // compute side: fragment offsets within a slice
    const int row_a = 16 * RW_CB * cw + lr, row_b = RW_CO + 16 * tw + lr;
    const int frag_a = row_a * 64 + 16 * lds_slot(row_a, lk);   // block c: + 16 c rows
    const int frag_b = row_b * 64 + 16 * lds_slot(row_b, lk);
    const int rnd = MODE == 0 && g.out_shift > 0 ? 1 << (g.out_shift - 1) : 0;

    // value k = 4 c + r of a lane: channel 16 (RW_CB cw + c) + 4 lk + r of tile
    // 16 tw + lr
    int P[RW_V][4], Q[RW_V][4], Z[RW_V][4];
    uint32_t out[4][RW_V];                                 // packed bytes
    // A finished output row i arrives value by value, v = its four pixels of
    // channel r of block c.  NHWC: word 4 c + j = channels r = 0..3 of pixel
    // (i, j), packed pair by pair; NCHW: word 4 c + r = the pixels of channel r.
    int prev[2][4];
    uint32_t half[2][4];
    uint32_t zmax = 0, in_row[4], in_col[4];               // MODE 1: masks of the lane's tile's pixels
    if constexpr (MODE == 1) {
        const long long tile = tl_blk + 16 * tw + lr;
        int img = 0, ty = 0, tx = 0;
        if (tile < g.ntiles) tile_coords(tile, g, img, ty, tx);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            in_row[i] = tile < g.ntiles && 4 * ty + i < g.h ? ~0u : 0u;
            in_col[i] = 4 * tx + i < g.w ? ~0u : 0u;
        }
    }
    auto put = [&](int i, int slot, int c, int r, const int (&v)[4]) __attribute__((always_inline)) {
        if constexpr (MODE == 1) {                         // channels past Cout hold zeros
#pragma unroll
            for (int j = 0; j < 4; ++j) zmax = max(zmax, (uint32_t)abs(v[j]) & in_row[i] & in_col[j]);
            asm volatile("" : "+v"(zmax));
            return;
        }
        if (LAYOUT == WINO_NCHW) {
            out[i][4 * c + r] = join2(requant2(v[0], v[1], g.out_shift), requant2(v[2], v[3], g.out_shift));
            asm volatile("" : "+v"(out[i][4 * c + r]));
            return;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (r == 0 || r == 2) prev[slot][j] = v[j];
            if (r == 1) half[slot][j] = requant2(prev[slot][j], v[j], g.out_shift);
            if (r == 3) {
                out[i][4 * c + j] = join2(half[slot][j], requant2(prev[slot][j], v[j], g.out_shift));
                asm volatile("" : "+v"(out[i][4 * c + j]));
            }
        }
    };
    // fold value 4 c + r of the finished row a of taps, accumulators m.  The
    // empty asm statements pin the results: they are read much later, and the
    // compiler would sink the folds past the next rows and keep all their
    // accumulators live.
    v4i bias_rnd;
    auto fold = [&](auto row_a, v4i (&m)[6][RW_CB], int c, int r) __attribute__((always_inline)) {
        constexpr int a = decltype(row_a)::value;
        const int k = 4 * c + r;
        int mv[6], z[4];
#pragma unroll
        for (int b = 0; b < 6; ++b) mv[b] = m[b][c][r] << g.tab.sh[6 * a + b];
        if (a == 1) {
            // bias plus rounding constant, injected through tap (1,1): its row
            // and column of A^T are all ones, so it reaches every output of
            // the tile once
            if (r == 0) bias_rnd = *(const v4i*)(bias_blk + 16 * (RW_CB * cw + c) + 4 * lk) + rnd;
            mv[1] += bias_rnd[r];
        }
        at_1d(mv, z);
        int y1[4], y2[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (a == 1 || a == 3) Z[k][j] = z[j];
            if (a == 2) {
                P[k][j] = Z[k][j] + z[j];
                Q[k][j] = Z[k][j] - z[j];
            }
            if (a == 4) {
                const int qv = Z[k][j] + z[j], rv = Z[k][j] - z[j];
                y1[j] = Q[k][j] + (rv << 1);
                y2[j] = P[k][j] + (qv << 2);
                P[k][j] += qv;
                Q[k][j] += rv << 3;
            }
            if (a == 0) P[k][j] += z[j];
            if (a == 5) Q[k][j] += z[j];
            if (a == 1 || a == 3) asm volatile("" : "+v"(Z[k][j]));
            if (a == 2 || a == 4) asm volatile("" : "+v"(P[k][j]), "+v"(Q[k][j]));
        }
        if (a == 4) {
            put(1, 0, c, r, y1);
            put(2, 1, c, r, y2);
        }
        if (a == 0) put(0, 0, c, r, P[k]);
        if (a == 5) put(3, 0, c, r, Q[k]);
    };

#pragma unroll
    for (int st = 0; st < C::NBUF - 1; ++st) {             // nstage >= NBUF
#pragma unroll
        for (int i = 0; i < C::G; ++i) issue_part(i);
        issue_end(st % C::SPR);
    }
    int s = 0, rd_off = 0;
    // One stage: taps G j .. G j + G - 1 of a row x 64 input channels into the
    // row's accumulators m (from zero if FIRST).  fold_b(b) folds part of the row
    // before by VALU instructions between this stage's MFMAs: both waves of a
    // SIMD are in the same phase, so a fold after the row's last stage would
    // leave the matrix cores idle.
    // COPY: the copies of stage s + NBUF - 1 go out (RW_COPY), or that depends
    // on s (RW_ASK).  Only the last rows have to ask, and without the branches a
    // stage is one block for the scheduler.
    auto stage = [&](auto first, auto part, auto copy, auto fold_b, v4i (&m)[6][RW_CB])
        __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first)::value;
        constexpr int COPY = decltype(copy)::value, J = decltype(part)::value;
        // stage s has landed once only the stages after it are pending:
        // NBUF - 2, less at the end
        const int later = nstage - 1 - s;
        if (COPY == RW_COPY || later >= C::NBUF - 2) {
            WINO_WAIT_VM_LDS((C::NBUF - 2) * C::LPW);
        } else {
            if (later >= 3) WINO_WAIT_VM_LDS(3 * C::LPW);
            else if (later == 2) WINO_WAIT_VM_LDS(2 * C::LPW);
            else if (later == 1) WINO_WAIT_VM_LDS(C::LPW);
            else WINO_WAIT_VM_LDS(0);
        }
        ring_barrier();   // stage s visible; stage s - 1, whose buffer is refilled, consumed
        // The copies go out one slice per tap, between the MFMAs: a copy
        // instruction holds its wave while the load path is busy (64 B/clk per
        // CU, 16 clk and more for each), and six in a row kept every wave of an
        // earlier version from computing for 400-700 clk.
        const bool more = COPY == RW_COPY || s + C::NBUF - 1 < nstage;
        const uint8_t* const base = lds + rd_off;
        rd_off = rd_off == (C::NBUF - 1) * C::STAGE ? 0 : rd_off + C::STAGE;
        ++s;
        // fragments of two taps in flight ahead of the MFMAs
        v4i fa[2][RW_CB], fb[2];
        auto frag = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < RW_CB; ++c)
                fa[b & 1][c] = *(const v4i*)(base + b * C::SLICE + frag_a + 1024 * c);
            fb[b & 1] = *(const v4i*)(base + b * C::SLICE + frag_b);
        };
        frag(0);
        frag(1);
        const v4i zero = (v4i){0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < C::G; ++b) {
            const int t = C::G * J + b;
#pragma unroll
            for (int c = 0; c < RW_CB; ++c)
                m[t][c] =
                    __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[b & 1][c], fb[b & 1], FIRST ? zero : m[t][c], 0, 0, 0);
            if (more) issue_part(b);
            if (b + 2 < C::G) frag(b + 2);
            fold_b(b);
            __builtin_amdgcn_sched_barrier(0);     // the taps' parts stay apart
        }
        if (more) issue_end((J + C::NBUF - 1) % C::SPR);
    };
    const std::true_type yes;
    const std::false_type no;
    // k-chunk 0 or 1 of a row, with its share of the row before (f(k) folds value
    // k): two values behind taps 1-4 of a row's only chunk, else one behind taps
    // 1-4 of the first two
    auto chunk = [&](auto first, auto half, v4i (&m)[6][RW_CB], auto cp, auto f) __attribute__((always_inline)) {
        constexpr int H = decltype(half)::value;
        auto at = [&](int t) __attribute__((always_inline)) {
            if (t < 1 || t > 4) return;
            if (ONE) {
                f(2 * t - 2);
                f(2 * t - 1);
            } else {
                f(4 * H + t - 1);
            }
        };
        stage(first, std::integral_constant<int, 0>{}, cp, [&](int b) __attribute__((always_inline)) { at(b); }, m);
        if constexpr (C::SPR == 2)
            stage(first, std::integral_constant<int, 1>{}, cp, [&](int b) __attribute__((always_inline)) { at(3 + b); }, m);
    };
    auto row = [&](v4i (&m)[6][RW_CB], auto cp, auto f) __attribute__((always_inline)) {
        auto none = [](int) __attribute__((always_inline)) {};
        chunk(yes, std::integral_constant<int, 0>{}, m, cp, f);
        if constexpr (!ONE) {
            chunk(no, std::integral_constant<int, 1>{}, m, cp, f);
            for (int kc = 2; kc < nkc; ++kc) chunk(no, std::integral_constant<int, 1>{}, m, cp, none);
        }
    };
    // with one k-chunk all of s is known at compile time; else a row has at
    // least 2 SPR stages, and a copy reaches NBUF - 1 stages ahead
    const std::integral_constant<int, ONE ? RW_ASK : RW_COPY> copy;
    const std::integral_constant<int, (ONE || C::NBUF - 1 > 2 * C::SPR) ? RW_ASK : RW_COPY> copy4;
    const std::integral_constant<int, RW_ASK> copy5;
    v4i ma[6][RW_CB], mb[6][RW_CB];
#define RW_ROW(m, cp, mp, prev) \
    row(m, cp,                  \
        [&](int k) __attribute__((always_inline)) { fold(std::integral_constant<int, prev>{}, mp, k >> 2, k & 3); })
    row(ma, copy, [](int) __attribute__((always_inline)) {});
    RW_ROW(mb, copy, ma, 1);
    RW_ROW(ma, copy, mb, 2);
    RW_ROW(mb, copy, ma, 3);
    RW_ROW(ma, copy4, mb, 4);
    RW_ROW(mb, copy5, ma, 0);
#undef RW_ROW
#pragma unroll
    for (int k = 0; k < RW_V; ++k) fold(std::integral_constant<int, 5>{}, mb, k >> 2, k & 3);
    if constexpr (MODE == 1) {
        __syncthreads();                                   // every wave is done reading the ring
        block_max<C::WAVES>(zmax, (uint32_t*)lds, (unsigned long long*)aux);
        return;
    }
    if (g.relu)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < RW_V; ++k) out[i][k] = relu4(out[i][k]);

    if constexpr (LAYOUT == WINO_NHWC) {
        // gather the block's output in LDS (the ring is idle now) so that
        // every pixel's 64 channel bytes leave together
        constexpr int PITCH = 16 * 64 + 16;   // bytes per tile; the pad spreads lanes over banks
        static_assert(C::TL * PITCH <= C::NBUF * C::STAGE, "output staging fits the ring");
        __syncthreads();                      // every wave is done reading the ring
        uint8_t* ot = lds + (16 * tw + lr) * PITCH + 16 * RW_CB * cw + 4 * lk;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < RW_CB; ++c)
#pragma unroll
                for (int j = 0; j < 4; ++j) *(uint32_t*)(ot + 64 * (4 * i + j) + 16 * c) = out[i][4 * c + j];
        __syncthreads();
        if (g.y_staged) {
            // wave w stores tiles w, w + WAVES, ...: lane = 16-byte quarter q of
            // pixel p; all LDS reads first, so that they overlap
            const int p = lane >> 2, q = lane & 3;
            constexpr int NT = C::TL / C::WAVES;
            v4i d[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i)
                d[i] = *(const v4i*)(lds + (wave + C::WAVES * i) * PITCH + 64 * p + 16 * q);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const long long tile = tl_blk + wave + C::WAVES * i;   // wave-uniform
                if (tile >= g.ntiles) break;
                int img, ty, tx;
                tile_coords(tile, g, img, ty, tx);
                const int yy = 4 * ty + (p >> 2), xx = 4 * tx + (p & 3);
                // non-temporal: the output is not read again here, and in L2
                // it would evict the operands the next round of blocks reads
                // (measured 2-3% of the kernel at C5 and C4)
                if (yy < g.h && xx < g.w)
                    __builtin_nontemporal_store(
                        d[i], (v4i*)(y + (((long long)img * g.h + yy) * g.w + xx) * g.cout + co_blk + 16 * q));
            }
        } else if ((g.cout & 3) == 0 && ((uintptr_t)y & 3) == 0) {
            // words of four channels: lane = word lane % 16 of pixel 4 k + lane / 16
            const int q = lane & 15;
            const bool co_ok = co_blk + 4 * q < g.cout;
            for (int tl = wave; tl < C::TL; tl += C::WAVES) {
                const long long tile = tl_blk + tl;
                if (tile >= g.ntiles) break;
                int img, ty, tx;
                tile_coords(tile, g, img, ty, tx);
                const int xx = 4 * tx + (lane >> 4);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (4 * ty + k < g.h && xx < g.w && co_ok)
                        *(uint32_t*)(y + (((long long)img * g.h + 4 * ty + k) * g.w + xx) * g.cout + co_blk + 4 * q) =
                            *(const uint32_t*)(lds + tl * PITCH + 64 * (4 * k + (lane >> 4)) + 4 * q);
            }
        } else {
            // any Cout and alignment: lane = channel, one pixel per store
            const int co = co_blk + lane;
            for (int tl = wave; tl < C::TL; tl += C::WAVES) {
                const long long tile = tl_blk + tl;
                if (tile >= g.ntiles) break;
                int img, ty, tx;
                tile_coords(tile, g, img, ty, tx);
                for (int p = 0; p < 16; ++p) {
                    const int yy = 4 * ty + (p >> 2), xx = 4 * tx + (p & 3);
                    if (yy < g.h && xx < g.w && co < g.cout)
                        y[(((long long)img * g.h + yy) * g.w + xx) * g.cout + co] =
                            (int8_t)lds[tl * PITCH + 64 * p + lane];
                }
            }
        }
    } else {
        const long long tile = tl_blk + 16 * tw + lr;
        if (tile >= g.ntiles) return;
        int img, ty, tx;
        tile_coords(tile, g, img, ty, tx);
        const bool word = (g.w & 3) == 0 && ((uintptr_t)y & 3) == 0;
#pragma unroll
        for (int c = 0; c < RW_CB; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int co = co_blk + 16 * (RW_CB * cw + c) + 4 * lk + r;
                if (co >= g.cout) continue;
                int8_t* base = y + (((long long)img * g.cout + co) * g.h + 4 * ty) * g.w + 4 * tx;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (4 * ty + i >= g.h) continue;
                    const uint32_t w = out[i][4 * c + r];
                    if (word) {
                        *(uint32_t*)(base + (long long)i * g.w) = w;
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (4 * tx + j < g.w) base[(long long)i * g.w + j] = (int8_t)(w >> (8 * j));
                    }
                }
            }
    }
}
