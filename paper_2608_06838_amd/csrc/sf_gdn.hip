// sf_gdn.hip -- gfx950 forward walk of the gated delta rule (Gated DeltaNet,
// the scalar-plus-low-rank transition of Sec. 2.1):
//
//   S_t = a_t (I - beta_t k_t k_t^T) S_{t-1} + beta_t k_t v_t^T,   o_t = S_t^T q_t,
//
// with S in R^{Dk x Dv} (the transpose of the paper's S) and a_t = exp(g_t).
//
// Chunkwise form (per chunk of C tokens, S the state entering it, b_t the
// chunk-local inclusive cumulative log-decay, gamma_t = e^{b_t}):
//   A[t][s]  = beta_t e^{b_t - b_s} (k_t . k_s)      for s < t   (strictly lower)
//   (I + A) [W | Ubar] = [diag(beta gamma) K | diag(beta) V]     (T = (I + A)^{-1} by blocks, then T R)
//   U        = Ubar - W S                                          (the corrected values, V^new)
//   O        = diag(gamma) Q S + (Q K^T o Gamma) U,  Gamma[t][s] = e^{b_t - b_s} (s <= t)
//   S_next   = gamma_C S + (K o e^{b_C - b})^T U
// This follows from writing u_t = beta_t (v_t - a_t S_{t-1}^T k_t), so that
// S_t = a_t S_{t-1} + k_t u_t^T is a plain gated linear recurrence in u, and
// solving the within-chunk dependence of u on the earlier u's.
//
// T = (I + A)^{-1} needs k, g and beta alone: k_gdn_tprep forms it for every
// chunk in parallel and the walks read it (D = 64 walks form it themselves).  One
// workgroup walks the chunks of one (batch, head) superchunk with the state in
// registers, each wave on its own state columns; with T given, U = T diag(beta)
// (V - diag(gamma) K S) needs no product shared between waves.  U, the output and
// the state update are MFMA products whose computed operands (S, T, P, U) go in
// as bf16 hi/lo pairs, straight from their accumulators where they are a wave's
// own.
//
// Superchunk parallelism (the Pre / ST / Out split of Sec. 2.2 with the delta
// rule's matrix-valued transition): the chunk map S -> gamma_C S + K~^T (Ubar - W S)
// is affine in S, so a superchunk of chunks maps S_J to S_{J+1} = M_J S_J + N_J
// with dense M_J, N_J in R^{Dk x Dk}, R^{Dk x Dv}.
//   k_gdn_walk<W_PREP>: walks the superchunk's chunks with the state M (from the
//     identity, V = 0) or N (from zero), one workgroup each.  No outputs.
//   k_gdn_scan: S_{J+1} = M_J S_J + N_J in fp32, sequential over J, 16 state
//     columns per workgroup; writes every S_J and S_out.
//   k_gdn_walk<W_OUT>: the output walk above from S_J over superchunk J;
//   k_gdn_walk<W_STORE>: the same walk without outputs, writing the state that
//     enters every chunk (for the backward).
#include "sf_chunk.hpp"

namespace sf {

namespace {

// 16x16x16 bf16 MFMA: A lane (q, n) holds row n, k = 4q .. 4q+3; B lane (q, n)
// holds k = 4q .. 4q+3 of column n; the accumulator holds rows 4q .. 4q+3 of
// column n, the same slots as a B operand.
typedef short s4v __attribute__((ext_vector_type(4)));
typedef int s4v2 __attribute__((ext_vector_type(4)));  // a 16-byte block
__device__ __forceinline__ void mma16(f32x4 &c, s4v a, s4v b) {
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
// hi = bf16(x), lo = bf16(x - hi), as the raw 16-bit patterns
__device__ __forceinline__ void split4(const f32x4 &x, s4v &hi, s4v &lo) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const __bf16 h = (__bf16)x[j];
        const __bf16 l = (__bf16)(x[j] - (float)h);
        hi[j] = __builtin_bit_cast(short, h);
        lo[j] = __builtin_bit_cast(short, l);
    }
}

// Column c of (I + M)^{-1} for a strictly lower 16 x 16 block M (row pitch ld) by
// forward substitution in fp32: x[r] = [r == c] - sum_{s < r} M[r][s] x[s].  Right-looking: once x[s]
// is final, every later row takes its term, so the 120 products form 16
// dependent steps of independent updates instead of one chain.  Each row's sum
// still runs over s in increasing order.
__device__ __forceinline__ void gdn_diag_column(const float *M, int ld, int c, float (&x)[16]) {
    float acc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int s2 = 0; s2 < 16; ++s2) {
        x[s2] = s2 == c ? 1.f : (s2 > c ? -acc[s2] : 0.f);
#pragma unroll
        for (int r = s2 + 1; r < 16; ++r) acc[r] = fmaf(M[r * ld + s2], x[s2], acc[r]);
    }
}
// The triangular 64 x 64 pair tiles of the walks (T, P, P^T as bf16 hi/lo) hold
// the three 32 x 32 quadrants that are not all zero, each 64-byte rows with
// their four 16-byte blocks XOR-swizzled by the row, hi then lo: 12 KB instead of
// the 20 of two padded square tiles, which is what lets two walk workgroups share
// a CU.  Quadrants (0,0), off-diagonal, (1,1) in that order, for a lower (r >= c)
// and an upper triangle alike; the all-zero 16 x 16 blocks inside the diagonal
// quadrants are stored.  SW: the swizzle for the way the rows are read, 0 for
// fragment rows arow(tt, n) (8 apart in fours), 1 for 16 consecutive rows.
constexpr int TRI = 3 * 32 * 32;  // elements of one half (hi or lo)
template <int SW>
__device__ __forceinline__ int tri_pos(int r, int c) {
    const int sw = SW ? (r >> 1) & 3 : ((r >> 1) & 1) | (((r >> 3) & 1) << 1);
    return ((r >> 5) + (c >> 5)) * 1024 + (r & 31) * 32 + ((((c & 31) >> 3) ^ sw) << 3) + (c & 7);
}

// T = (I + A)^{-1} (A in sA, pitch C + 4) as the bf16 hi/lo pair that every
// consumer splits it into (tri_pos<0>, raw 16-bit patterns): the four diagonal
// blocks by forward substitution in fp32 (64 threads, one column each), the
// off-diagonal blocks level by level (i - j = 1, 2, 3; wave j forms T_ij = -T_ii
// sum_{k=j}^{i-1} A_ik T_kj on 16x16x16 MFMA, the inner sum staying in its
// accumulator, which is already the B operand of the T_ii product).
// (A diagonal block N is nilpotent, and (I + N)^{-1} = (I + N^8)(I + N^4)
// (I + N^2)(I - N) on MFMA is faster; but the series' partial sums grow like
// binomial coefficients when neighbouring keys are nearly parallel with little
// decay, and the outputs then lost up to 1e-1 (bf16 hi/lo operands) or 1e-3
// (fp32 MFMA) against the oracle, where substitution keeps them at output
// rounding.)  Four waves; ends with a barrier.
__device__ __forceinline__ void gdn_tinv_hl(int tid, const float *sA, short *sTh, short *sTl) {
    constexpr int LA = C + 4;
    const int w = tid >> 6, lane = tid & 63, q4 = lane >> 4, n16 = lane & 15;
    if (tid < 64) {  // one column of a diagonal block per thread
        const int o = 16 * (tid >> 4), c = tid & 15;
        float x[16];
        gdn_diag_column(sA + o * LA + o, LA, c, x);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const __bf16 h = (__bf16)x[r];
            const int p = tri_pos<0>(o + r, o + c);
            sTh[p] = __builtin_bit_cast(short, h);
            sTl[p] = __builtin_bit_cast(short, (__bf16)(x[r] - (float)h));
        }
    } else if (tid < 192) {  // the zero blocks (0,1) and (2,3) of the diagonal quadrants
        const int e = tid - 64, b = e >> 6, r = 32 * b + ((e >> 2) & 15), c = 32 * b + 16 + 4 * (e & 3);
        *reinterpret_cast<s4v *>(&sTh[tri_pos<0>(r, c)]) = s4v{0, 0, 0, 0};
        *reinterpret_cast<s4v *>(&sTl[tri_pos<0>(r, c)]) = s4v{0, 0, 0, 0};
    }
    __syncthreads();
#pragma unroll
    for (int d = 1; d < 4; ++d) {
        if (w < 4 - d) {  // block (i, j) = (d + w, w)
            const int i = d + w, j = w;
            f32x4 y = {0.f, 0.f, 0.f, 0.f};
            for (int k = j; k < i; ++k) {
                const f32x4 av = *reinterpret_cast<const f32x4 *>(&sA[(16 * i + n16) * LA + 16 * k + 4 * q4]);
                s4v ah, al, bh = {0, 0, 0, 0}, bl = bh;
                split4(av, ah, al);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int p = tri_pos<0>(16 * k + 4 * q4 + u, 16 * j + n16);
                    bh[u] = sTh[p];
                    bl[u] = sTl[p];
                }
                mma16(y, ah, bh);
                mma16(y, ah, bl);
                mma16(y, al, bh);
            }
            const int p = tri_pos<0>(16 * i + n16, 16 * i + 4 * q4);
            const s4v th = *reinterpret_cast<const s4v *>(&sTh[p]);
            const s4v tl = *reinterpret_cast<const s4v *>(&sTl[p]);
            s4v yh, yl, h, l;
            split4(y, yh, yl);
            f32x4 t = {0.f, 0.f, 0.f, 0.f};
            mma16(t, th, yh);
            mma16(t, th, yl);
            mma16(t, tl, yh);
            split4(-t, h, l);
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // rows 16i + 4 q4 + r of column 16j + n16
                const int p2 = tri_pos<0>(16 * i + 4 * q4 + r, 16 * j + n16);
                sTh[p2] = h[r];
                sTl[p2] = l[r];
            }
        }
        __syncthreads();
    }
}

// A[t][s] = beta_t e^{b_t - b_s} k_t.k_s (s < t) of a staged chunk on the causal
// tiles, 10 over the four waves, into sA (fp32, pitch C + 4)
template <typename T, int D, int LDN, int SWX>
__device__ __forceinline__ void gdn_a_scores(int w, int lane, const T *sK, const float *sb, const float *sbeta, float *sA) {
    constexpr int LDA = C + 4;
    const int q4 = lane >> 4, n16 = lane & 15;
    const LaneOff swo = swz_off<T, LDN, SWX>(lane);
    for (int i = w; i < 10; i += 4) {
        int tt, st;
        tri_tile(i, tt, st);
        f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks)
            mma(p, ldfrag_swz<T, LDN, SWX>(sK, swo, 16 * st, 32 * ks), ldfrag_swz<T, LDN, SWX>(sK, swo, 16 * tt, 32 * ks));
        const int t = 16 * tt + n16;
        const float bt = sb[t], be = sbeta[t];
        const f32x4 bs = *reinterpret_cast<const f32x4 *>(&sb[16 * st + 4 * q4]);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = 16 * st + 4 * q4 + r < t ? be * p[r] * fexp2(bt - bs[r]) : 0.f;
        *reinterpret_cast<f32x4 *>(&sA[t * LDA + 16 * st + 4 * q4]) = v;
    }
}

// T of every chunk, all chunks in parallel, into the rows of an output tensor
// that a later kernel overwrites (o forward, dq backward): token row t of the
// chunk holds T[t][0..63] hi, then lo, 256 bytes (so D = 128 only; the walks of
// D = 64 form T themselves).  T depends on k, g and beta alone, and its
// substitution is a serial chain: inside the walks it was half of every chunk's
// latency, and each pass of the backward formed it again.  Here four workgroups
// per CU (36 KB of LDS) hide the chain of one behind the others'.
template <typename T, int D>
__global__ void __launch_bounds__(256) k_gdn_tprep(GdnArgs a) {
    static_assert(D == 128 && sizeof(T) == 2, "T's pair fills a row of 128 bf16");
    constexpr int LDN = D + pad<T>(), SWX = swx<T, D>();
    __shared__ __attribute__((aligned(16))) T sK[C * LDN];  // then T's pair
    __shared__ __attribute__((aligned(16))) float sA[C * (C + 4)];
    __shared__ __attribute__((aligned(16))) float sb[C], sbeta[C];
    static_assert(2 * TRI <= C * LDN, "T's pair fits the key tile");
    short *const sTh = reinterpret_cast<short *>(sK), *const sTl = sTh + TRI;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nc = (int)(a.L / C), bh = blockIdx.x / nc, c = blockIdx.x % nc, bb = bh / a.H, hh = bh % a.H;
    const int64_t xo = bb * a.sx_b + hh * a.sx_h + (int64_t)c * C * a.sx_l;
    const int64_t go = bb * a.sg_b + hh * a.sg_h + (int64_t)c * C * a.sg_l;
    Tile<T, D, 256> t;
    t.load((const T *)a.k + xo, a.sx_l, tid);
    if (w == 0) {
        sb[lane] = wave_scan_dpp(a.g[go + lane * a.sg_l] * LOG2E);
        sbeta[lane] = a.beta[go + lane * a.sg_l];
    }
    t.store_swz(sK, LDN, tid, SWX);
    __syncthreads();
    gdn_a_scores<T, D, LDN, SWX>(w, lane, sK, sb, sbeta, sA);
    __syncthreads();
    gdn_tinv_hl(tid, sA, sTh, sTl);
    T *out = (T *)a.tw + xo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // 16-byte blocks: row u / 16, then hi 0-7, lo 0-7
        const int u = 256 * i + tid, r = u >> 4, j = u & 15, cc = 8 * (j & 7);
        if (r < 32 && cc >= 32) continue;  // the zero quadrant, never read
        *reinterpret_cast<s4v2 *>(out + r * a.sx_l + 8 * j) =
            *reinterpret_cast<const s4v2 *>((j < 8 ? sTh : sTl) + tri_pos<0>(r, cc));
    }
}

enum { W_OUT = 0, W_PREP = 1, W_STORE = 2 };

// Registers and LDS of the walks.  D = 128: four waves of two 16-column tiles
// each, so every shared operand fragment read from LDS feeds both, and two
// workgroups per CU (<= 256 registers, <= 80 KB of LDS) cover each other's
// barriers.  D = 64: four waves of one tile.  Column n of tile m is channel
// 32w + 8 (n / 4) + 4m + n % 4 (two tiles), so that a lane's output rows of the
// two tiles are 8 consecutive channels, one 16-byte store.
template <int D>
struct GdnCols {
    static constexpr int NCT = D / 64;
    int c0, n16;
    __device__ __forceinline__ int col(int m) const { return NCT == 2 ? c0 + 8 * (n16 >> 2) + 4 * m + (n16 & 3) : c0 + n16; }
    __device__ __forceinline__ int base(int m) const { return c0 + 4 * m; }  // ldfragTR column of tile m
};

// A D x D fp32 state in the walks' register layout (slot [m][i][r] = row
// prow(i, r), column col(m)) through a buffer resource: one lane offset, the rest
// of the address uniform (64 flat addresses would spill).
template <int D>
struct StateIO {
    static constexpr int NCT = GdnCols<D>::NCT, NK = D / 16;
    uint32_t off;
    __device__ __forceinline__ StateIO(const GdnCols<D> &cl, int q4) : off((uint32_t)(8 * q4 * D + cl.col(0)) * 4) {}
    __device__ __forceinline__ static uint32_t at(int m, int i, int r) {
        return (uint32_t)((32 * (i >> 1) + 4 * (i & 1) + r) * D + 4 * m) * 4;
    }
    __device__ __forceinline__ void load(f32x4 (&S)[NCT][NK], const float *src) const {
        const rsrc_t rs = buf_rsrc(src, D * D * 4);
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int i = 0; i < NK; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) S[m][i][r] = buf_ld<float>(rs, off, at(m, i, r));
    }
    __device__ __forceinline__ void store(const f32x4 (&S)[NCT][NK], float *dst) const {
        const rsrc_t rs = buf_rsrc(dst, D * D * 4);
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int i = 0; i < NK; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) buf_st(rs, off, at(m, i, r), S[m][i][r]);
    }
};

// The fragment reads' positions in a triangular tile are one lane offset plus a
// constant (the swizzle does not see the tile index); spelled out, since the
// compiler would keep every position in a register of its own.
//   rows ar + roff(tt), columns 32 ks + 8 q4 ..   (tri_pos<0>, base ar, 8 q4)
__device__ __forceinline__ constexpr int tri_a(int tt, int ks) { return ((tt >> 1) + ks) * 1024 + 4 * (tt & 1) * 32; }
//   rows 16 tt + n16, columns 32 ks + 8 q4 ..     (tri_pos<1>, base n16, 8 q4)
__device__ __forceinline__ constexpr int tri_b(int tt, int ks) { return ((tt >> 1) + ks) * 1024 + 16 * (tt & 1) * 32; }

// A chunk's state as the hi/lo pair that the products split it into, transposed:
// two [v][k] planes of bf16 (the bytes of the fp32 state), written by the wave that
// splits it anyway, a fragment per 16-byte store, and read by the per-chunk
// gradients as fragments, with no splitting there.  Fragment ks of tile m: column
// col(m), rows 32 ks + 8 q4 ..
template <typename T, int D>
__device__ __forceinline__ void put_state_pair(rsrc_t rs, uint32_t off, int m, int ks, const frag_t<T> &h, const frag_t<T> &l) {
    buf_st(rs, off, (uint32_t)(4 * m * D + 32 * ks) * 2, h);
    buf_st(rs, off, (uint32_t)(4 * m * D + 32 * ks + D * D) * 2, l);
}

// the 16-byte blocks of T's pair that this thread moves between the rows of the
// tensor that holds it and LDS (see k_gdn_tprep): row 16 i + tid / 16, block tid % 16
template <typename T>
struct TriTile {
    s4v2 r[4];
    __device__ __forceinline__ void load(rsrc_t rs, uint32_t off, uint32_t step, int tid) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i >= 2 || (tid & 7) < 4) r[i] = buf_ld<s4v2>(rs, off, i * step);
    }
    __device__ __forceinline__ static int base(int tid) { return ((tid & 8) ? TRI : 0) + tri_pos<0>(tid >> 4, 8 * (tid & 7)); }
    __device__ __forceinline__ void store(short *t, int base, int tid) const {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i >= 2 || (tid & 7) < 4) *reinterpret_cast<s4v2 *>(t + base + (i >> 1) * 1024 + (i & 1) * 512) = r[i];
    }
};

// A chunk tile copied from memory straight into LDS, 1 KB per wave and
// instruction (lane l's 16 bytes to base + 16 l), without passing registers: rows
// of D bf16 unpadded, the 16-byte blocks of row r XOR-swizzled by f(r) = (r % 8) ^
// 4 (r / 8 % 2) through the source addresses, so that fragment reads over 16 rows
// (and the transposing ones over rows 8 apart) touch every bank once.
template <typename T, int D, int NW>
struct DmaTile {
    static constexpr int BPR = D / 8, RPI = 64 / BPR, NI = C / RPI / NW;  // blocks per row, rows per instruction
    uint32_t v0, v1;  // source offsets; v1 for the instructions whose rows flip f's bit 2 (chosen as in LaneOff::at)
    __device__ __forceinline__ DmaTile(int lane, int64_t ld) {
        const int r = lane / BPR, b = (lane % BPR) ^ r;  // r < RPI <= 8: f(r) = r
        v0 = (uint32_t)((r * ld + 8 * b) * (int64_t)sizeof(T));
        v1 = (uint32_t)((r * ld + 8 * (b ^ 4)) * (int64_t)sizeof(T));
    }
    __device__ __forceinline__ void issue(rsrc_t rs, T *lds, int w, uint32_t row_bytes) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int k = NI * w + i;
            const bool flip = (D == 128 ? k ^ (k >> 1) : k) & 1;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + 512 * k), 16,
                                                     v0 + (flip ? v1 - v0 : 0), (int)(RPI * k * row_bytes), 0, 0);
        }
    }
    // fragment rows 16 tt + n16, columns 32 ks + 8 q4: base[ks & 1] + row0 D + 64 (ks >> 1)
    __device__ __forceinline__ static void row_base(int lane, int (&o)[2]) {
        const int q = lane >> 4, n = lane & 15, f = (n & 7) ^ (((n >> 3) & 1) << 2);
        o[0] = n * D + 8 * (q ^ f);
        o[1] = n * D + 8 * (q ^ 4 ^ f);
    }
};
// T's packed pair the same way (tri_pos<0>): 12 instructions, three per wave
struct DmaTri {
    uint32_t v;
    __device__ __forceinline__ DmaTri(int lane, int64_t ld) {
        const int r = lane >> 2, sw = ((r >> 1) & 1) | (((r >> 3) & 1) << 1);
        v = (uint32_t)(r * ld * 2 + 16 * ((lane & 3) ^ sw));
    }
    __device__ __forceinline__ void issue(rsrc_t rs, short *lds, int w, uint32_t row_bytes) const {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int k = 3 * w + i, h = k / 6, qd = (k % 6) >> 1, rows = 16 * (k & 1) + (qd > 0 ? 32 : 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + 512 * k), 16, v,
                                                     (int)(rows * row_bytes) + h * 128 + (qd == 2 ? 64 : 0), 0, 0);
        }
    }
};

// The forward walks.  Per chunk, each wave on its own state columns:
//   X = V - gamma o (K S),   U = T (beta o X),   O = gamma o (Q S) + P U,
//   S = gamma_C S + K^T (e^{b_C - b} o U)
// (U = Ubar - W S with the products regrouped: K enters exactly, S and X as hi/lo
// pairs, and neither W nor Ubar is formed).  V joins X's accumulators through an
// MFMA with the identity, which is exact and needs no 2-byte LDS reads.  Nothing
// but P and the staged tiles is shared between waves, so a chunk has two barriers
// (three with P).  TPRE: T comes from k_gdn_tprep; else the walk forms it (D = 64, and
// D = 128 for forward calls of one chunk, which are two launches otherwise).
template <typename T, int D, int MODE, bool TPRE = D == 128>
__global__ void __launch_bounds__(256, 2) k_gdn_walk(GdnArgs a) {
    constexpr bool PREP = MODE == W_PREP, OUTP = MODE == W_OUT;  // STORE: states only
    constexpr int NT = 256, NK = D / 16, NCT = GdnCols<D>::NCT;
    constexpr int LDN = D + pad<T>(), SWX = swx<T, D>(), LDA = C + 4;
    __shared__ __attribute__((aligned(16))) T sQ[OUTP ? C * D : 8];    // DmaTile
    __shared__ __attribute__((aligned(16))) T sK[C * LDN];             // swizzled
    __shared__ __attribute__((aligned(16))) T sV[C * LDN];             // swizzled
    __shared__ __attribute__((aligned(16))) short sT[2 * TRI];         // T, hi then lo
    __shared__ __attribute__((aligned(16))) T sP[OUTP ? 2 * TRI : 8];  // P[t][s] = e^{b_t-b_s} q_t.k_s, hi then lo
    __shared__ __attribute__((aligned(16))) float sA[TPRE ? 4 : C * LDA];
    __shared__ __attribute__((aligned(16))) float sb[C], sq[C], se[C], sbeta[C];

    const int tid = threadIdx.x, lane = tid & 63, q4 = lane >> 4, n16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const GdnCols<D> cl{16 * NCT * w, n16};
    // items: (b, h, J) with J < n_super (walk) or J < n_prep (prep).  The prep's M
    // (role 0) and N (role 1) are walks of their own, 8 apart in dispatch order (one XCD).
    const int nJ = PREP ? a.n_prep : a.n_super;
    int item = blockIdx.x, role = 1;
    if constexpr (PREP) {
        role = (item >> 3) & 1;
        item = (item >> 4) * 8 + (item & 7);
        if (item >= a.B * a.H * nJ) return;
    }
    const int bh = item / nJ, J = item % nJ;
    const int bb = bh / a.H, hh = bh % a.H;
    const int64_t tok0 = (int64_t)J * a.ts;
    const int64_t xo = bb * a.sx_b + hh * a.sx_h + tok0 * a.sx_l;
    const T *Q = (const T *)a.q + xo;
    const T *K = (const T *)a.k + xo;
    const T *V = (const T *)a.v + xo;
    const T *TW = TPRE ? (const T *)a.tw + xo : nullptr;
    T *Y = (T *)a.o + xo;
    T *VN = OUTP && a.v_new ? (T *)a.v_new + xo : nullptr;
    const int64_t go = bb * a.sg_b + hh * a.sg_h + tok0 * a.sg_l;
    const float *gp = a.g + go;
    const float *bp = a.beta + go;
    const int64_t SS = (int64_t)D * D;
    const int nch = (int)((a.L - tok0 < a.ts ? a.L - tok0 : a.ts) / C);
    const LaneOff swo = swz_off<T, LDN, SWX>(lane), tro8 = tr_off8<T, LDN, SWX>(lane);
    const LaneOff tro = NCT == 2 ? tro8 : tr_off<T, LDN, SWX>(lane);  // this wave's own columns
    // Accumulator pairs (2m, 2m+1) of the state (rows: key channels) and of X, U
    // (rows: tokens) hold, in lane row q4, indices 32m + 8 q4 .. +7 (slot r of
    // tile i: prow(i, r)), so each pair splits into an operand fragment in plain
    // order with no lane swaps.  The products that build them read their A rows
    // in that order: fragment row n of tile i is arow(i, n).
    auto prow = [&](int i, int r) { return 32 * (i >> 1) + 8 * q4 + 4 * (i & 1) + r; };
    const int ar = 8 * (n16 >> 2) + (n16 & 3);                      // arow(i, n16) = ar + roff(i)
    auto roff = [](int i) { return 32 * (i >> 1) + 4 * (i & 1); };  // (also ldfragTR's column for tro8)
    const LaneOff ko = {ar * LDN + 8 * q4 + ((n16 >> 2) & 1) * SWX, ar * LDN + 8 * q4 - ((n16 >> 2) & 1) * SWX};
    const int ta = tri_pos<0>(ar, 8 * q4), pb = tri_pos<1>(n16, 8 * q4);
    // identity fragments: row arow(tt, n16) of tile tt against its own 32 tokens
    frag_t<T> eye[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 8; ++j) eye[h][j] = (T)(q4 == (n16 >> 2) && j == 4 * h + (n16 & 3) ? 1.f : 0.f);

    // S[m][i][r] = S[prow(i, r)][col(m)]: the walk's state starts from S_J (S_in for
    // one superchunk); the prep's M from I and its N from 0
    const float *src = a.n_super == 1 ? a.S_in + (a.S_in ? bh * SS : 0) : a.wsS + (int64_t)item * SS;
    const StateIO<D> sio(cl, q4);
    f32x4 S[NCT][NK];
#pragma unroll
    for (int m = 0; m < NCT; ++m)
#pragma unroll
        for (int i = 0; i < NK; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[m][i][r] = PREP && role == 0 && prow(i, r) == cl.col(m) ? 1.f : 0.f;
    if (!PREP && (a.n_super > 1 || a.S_in)) sio.load(S, src);

    using TT = Tile<T, D, NT>;
    TT t2, t3;
    const DmaTile<T, D, 4> dq(lane, a.sx_l);
    const DmaTri dt(lane, a.sx_l);
    const uint32_t rowb = (uint32_t)(a.sx_l * (int64_t)sizeof(T));
    int qb[2];
    DmaTile<T, D, 4>::row_base(lane, qb);
    TriTile<T> t4;
    float gl = 0.f, bl = 0.f;  // wave 3's: a load of a chunk's gates touches 64 cache lines
    const int64_t cstep = (int64_t)C * a.sx_l;
    const uint32_t cspan = chunk_span<T, D>(a.sx_l), gspan = (uint32_t)(((C - 1) * a.sg_l + 1) * 4);
    uint32_t toff[TT::RPT];
    TT::offsets(toff, a.sx_l, tid);
    const uint32_t goff = (uint32_t)(lane * a.sg_l * 4);
    const uint32_t tstep = (uint32_t)(16 * a.sx_l * (int64_t)sizeof(T));
    const int t4base = TriTile<T>::base(tid);
    const uint32_t t4off = (uint32_t)(((tid >> 4) * a.sx_l + 8 * (tid & 15)) * (int64_t)sizeof(T));
    const uint32_t voff = (uint32_t)((n16 * a.sx_l + cl.c0 + 4 * NCT * q4) * (int64_t)sizeof(T));
    const uint32_t coff = (uint32_t)(cl.col(0) * D + 8 * q4) * 2;  // chunk state pairs
    auto issue = [&](int c) {
        const int64_t nx = c * cstep;
        t2.load_buf(buf_rsrc(K + nx, cspan), toff, 0);
        if constexpr (TPRE && !OUTP) t4.load(buf_rsrc(TW + nx, cspan), t4off, tstep, tid);
        if (w == 3) {
            gl = buf_ld<float>(buf_rsrc(gp + (int64_t)c * C * a.sg_l, gspan), goff, 0);
            bl = buf_ld<float>(buf_rsrc(bp + (int64_t)c * C * a.sg_l, gspan), goff, 0);
        }
        if (!PREP || role) t3.load_buf(buf_rsrc(V + nx, cspan), toff, 0);
        if constexpr (OUTP) dq.issue(buf_rsrc(Q + nx, cspan), sQ, w, rowb);
        if constexpr (OUTP && TPRE) dt.issue(buf_rsrc(TW + nx, cspan), sT, w, rowb);
    };
    if (nch > 0) issue(0);

    const unsigned par = pair_parity(a.n_cu);
    for (int c = 0; c < nch; ++c) {
        pair_turn(par);
        if constexpr (OUTP) vm_wait_all();  // this wave's part of Q and T is in LDS
        __syncthreads();  // the previous chunk is done with every LDS tile
        t2.store_swz(sK, LDN, tid, SWX);
        if (!PREP || role) t3.store_swz(sV, LDN, tid, SWX);
        if constexpr (TPRE && !OUTP) t4.store(sT, t4base, tid);
        if (w == 3) {
            const float b2 = wave_scan_dpp(gl * LOG2E);
            const float b63 = lane_value(b2, 63);
            sb[lane] = b2;
            sq[lane] = fexp2(b2);
            se[lane] = fexp2(b63 - b2);
            sbeta[lane] = bl;
        }
        __syncthreads();

        if constexpr (OUTP) {  // P on the causal tiles
            for (int i = w; i < 10; i += 4) {
                int tt, st;
                tri_tile(i, tt, st);
                f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < D / 32; ++ks)
                    mma(p, ldfrag_swz<T, LDN, SWX>(sK, swo, 16 * st, 32 * ks), *reinterpret_cast<const frag_t<T> *>(&sQ[qb[ks & 1] + 16 * tt * D + 64 * (ks >> 1)]));
                const int t = 16 * tt + n16;
                const float bt = sb[t];
                const f32x4 bs = *reinterpret_cast<const f32x4 *>(&sb[16 * st + 4 * q4]);
                float v4[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v4[r] = 16 * st + 4 * q4 + r <= t ? p[r] * fexp2(bt - bs[r]) : 0.f;
                const int o = tri_pos<1>(t, 16 * st + 4 * q4);
                st4_split<T, true>(&sP[o], &sP[TRI + o], v4);
            }
            if (tid < 128) {  // the zero blocks (0,1) and (2,3) of the diagonal quadrants
                const int b = tid >> 6, o = tri_pos<1>(32 * b + ((tid >> 2) & 15), 32 * b + 16 + 4 * (tid & 3));
                *reinterpret_cast<s4v *>(&sP[o]) = s4v{0, 0, 0, 0};
                *reinterpret_cast<s4v *>(&sP[TRI + o]) = s4v{0, 0, 0, 0};
            }
        }
        if constexpr (!TPRE) {
            gdn_a_scores<T, D, LDN, SWX>(w, lane, sK, sb, sbeta, sA);
            __syncthreads();
            gdn_tinv_hl(tid, sA, sT, sT + TRI);
        }

        // X[t][v] = V[t][v] - gamma_t sum_k K[t][k] S[k][v] (rows t = prow(tt, r));
        // O^T[v][t] = sum_k S[k][v] Q[t][k]
        const rsrc_t rc = buf_rsrc(MODE == W_STORE ? a.wsSc + ((int64_t)bh * (a.L / C) + tok0 / C + c) * SS : nullptr, D * D * 4);
        f32x4 X[NCT][4], O[NCT][4];
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) X[m][tt] = O[m][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
            frag_t<T> fh[NCT], fl[NCT];
#pragma unroll
            for (int m = 0; m < NCT; ++m) {
                split_acc<T, true>(S[m][2 * ks], S[m][2 * ks + 1], fh[m], fl[m]);
                if constexpr (MODE == W_STORE) put_state_pair<T, D>(rc, coff, m, ks, fh[m], fl[m]);
            }
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const frag_t<T> kf = *reinterpret_cast<const frag_t<T> *>(
                    &sK[(((32 * ks) & SWX) ? ko.hi : ko.lo) + roff(tt) * LDN + 32 * ks]);
#pragma unroll
                for (int m = 0; m < NCT; ++m) {
                    mma(X[m][tt], kf, fh[m]);
                    mma(X[m][tt], kf, fl[m]);
                }
                if constexpr (OUTP) {
                    const frag_t<T> qf = *reinterpret_cast<const frag_t<T> *>(&sQ[qb[ks & 1] + 16 * tt * D + 64 * (ks >> 1)]);
#pragma unroll
                    for (int m = 0; m < NCT; ++m) mma2<T, true>(O[m][tt], fh[m], fl[m], qf);
                }
            }
            if constexpr (OUTP) sched_fence();
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const f32x4 gq = *reinterpret_cast<const f32x4 *>(&sq[prow(tt, 0)]);
#pragma unroll
            for (int m = 0; m < NCT; ++m) X[m][tt] *= -gq;
        }
        if (!PREP || role) {
#pragma unroll
            for (int ks = 0; ks < C / 32; ++ks)
#pragma unroll
                for (int m = 0; m < NCT; ++m) {
                    const frag_t<T> vf = ldfragTR<T, LDN, SWX>(sV, tro, 32 * ks, cl.base(m));
                    mma(X[m][2 * ks], eye[0], vf);
                    mma(X[m][2 * ks + 1], eye[1], vf);
                }
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const f32x4 be = *reinterpret_cast<const f32x4 *>(&sbeta[prow(tt, 0)]);
#pragma unroll
            for (int m = 0; m < NCT; ++m) X[m][tt] *= be;
        }
        if constexpr (OUTP) sched_fence();
        // U = T (beta o X)
        f32x4 U[NCT][4];
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) U[m][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            frag_t<T> xh[NCT], xl[NCT];
#pragma unroll
            for (int m = 0; m < NCT; ++m) split_acc<T, true>(X[m][2 * ks], X[m][2 * ks + 1], xh[m], xl[m]);
#pragma unroll
            for (int tt = 2 * ks; tt < 4; ++tt) {
                const frag_t<T> th = *reinterpret_cast<const frag_t<T> *>(&sT[ta + tri_a(tt, ks)]);
                const frag_t<T> tl = *reinterpret_cast<const frag_t<T> *>(&sT[ta + TRI + tri_a(tt, ks)]);
#pragma unroll
                for (int m = 0; m < NCT; ++m) {
                    mma(U[m][tt], th, xh[m]);
                    mma(U[m][tt], th, xl[m]);
                    mma(U[m][tt], tl, xh[m]);
                }
            }
        }
        if constexpr (OUTP) {
            __syncthreads();  // P is complete
            sched_fence();
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const float gt = sq[16 * tt + n16];
#pragma unroll
                for (int m = 0; m < NCT; ++m) O[m][tt] *= gt;
            }
#pragma unroll
            for (int ks = 0; ks < C / 32; ++ks) {
                frag_t<T> uh[NCT], ul[NCT];
#pragma unroll
                for (int m = 0; m < NCT; ++m) split_acc<T, true>(U[m][2 * ks], U[m][2 * ks + 1], uh[m], ul[m]);
#pragma unroll
                for (int tt = 2 * ks; tt < 4; ++tt) {
                    const frag_t<T> ph = *reinterpret_cast<const frag_t<T> *>(&sP[pb + tri_b(tt, ks)]);
                    const frag_t<T> pl = *reinterpret_cast<const frag_t<T> *>(&sP[pb + TRI + tri_b(tt, ks)]);
#pragma unroll
                    for (int m = 0; m < NCT; ++m) {
                        mma(O[m][tt], uh[m], ph);
                        mma(O[m][tt], uh[m], pl);
                        mma(O[m][tt], ul[m], ph);
                    }
                }
            }
            // V^new (optional): U[prow(tt, r)][col(m)]
            if (VN) {
                typedef short s1;
                const rsrc_t rn = buf_rsrc(VN + c * cstep, cspan);
                const uint32_t no = (uint32_t)((8 * q4 * a.sx_l + cl.col(0)) * (int64_t)sizeof(T));
#pragma unroll
                for (int m = 0; m < NCT; ++m)
#pragma unroll
                    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            __builtin_amdgcn_raw_buffer_store_b16(
                                __builtin_bit_cast(s1, cvt<T>(U[m][tt][r])), rn, no,
                                (uint32_t)(((roff(tt) + r) * a.sx_l + 4 * m) * (int64_t)sizeof(T)), 0);
            }
        }
        if constexpr (OUTP) {  // lane (q4, n16): channels c0 + 4 NCT q4 .. of token 16 tt + n16
            const rsrc_t ro = buf_rsrc(Y + c * cstep, cspan);
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                if constexpr (NCT == 2) {
                    typedef T v8 __attribute__((ext_vector_type(8)));
                    v8 o = {};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        o[r] = cvt<T>(O[0][tt][r]);
                        o[4 + r] = cvt<T>(O[1][tt][r]);
                    }
                    buf_st(ro, voff, tt * tstep, o);
                } else {
                    st4_buf<T>(ro, voff, tt * tstep, O[0][tt]);
                }
            }
        }
        if constexpr (OUTP) sched_fence();
        if (c + 1 < nch) issue(c + 1);

        // S = gamma_C S + K^T (e^{b_C - b} o U)
        const float gam = sq[C - 1];
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int i = 0; i < NK; ++i) S[m][i] *= gam;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const f32x4 ev = *reinterpret_cast<const f32x4 *>(&se[prow(tt, 0)]);
#pragma unroll
            for (int m = 0; m < NCT; ++m) U[m][tt] *= ev;
        }
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            frag_t<T> uh[NCT], ul[NCT];
#pragma unroll
            for (int m = 0; m < NCT; ++m) split_acc<T, true>(U[m][2 * ks], U[m][2 * ks + 1], uh[m], ul[m]);
#pragma unroll
            for (int i = 0; i < NK; ++i) {
                const frag_t<T> kf = ldfragTR<T, LDN, SWX>(sK, tro8, 32 * ks, roff(i));
#pragma unroll
                for (int m = 0; m < NCT; ++m) mma2b<T, true>(S[m][i], kf, uh[m], ul[m]);
            }
        }
    }
    // prep: M_J or N_J; walk: S_out after the last superchunk
    if (PREP || (OUTP && J == a.n_super - 1 && !(a.scan_out && a.n_super > 1))) {
        sio.store(S, PREP ? (role == 0 ? a.wsM : a.wsN) + (int64_t)item * SS : a.S_out + bh * SS);
    }
}

// (batch, head) and columns of a scan workgroup: the D / 16 column blocks of a head
// are 8 apart in dispatch order, on one XCD, whose L2 then reads the head's maps
// once for all of them
template <int D>
__device__ __forceinline__ bool scan_item(const GdnArgs &a, int &bh, int &col0) {
    const int x = blockIdx.x, r = x % (D / 2);
    bh = x / (D / 2) * 8 + r % 8;
    col0 = 16 * (r / 8);
    return bh < a.B * a.H;
}
template <int D>
dim3 scan_grid(unsigned bh) { return dim3((bh + 7) / 8 * (D / 2)); }

// S_{J+1} = M_J S_J + N_J for J = 0 .. n_super - 2 in fp32, S_0 = S_in (or 0);
// writes S_J (J < n_super) to wsS; with scan_out (maps of every superchunk)
// one more step gives S_out.  Workgroup (b, h, 16-column block), D / 16 waves;
// wave w owns the rows [16w, 16w + 16) of the block on the fp32 MFMA (16x16x4,
// fp32 products and sums): slot (j, u) of the contraction is k = 32 (j / 2) + 8 q4 +
// 4 (j % 2) + u on both sides, so a lane's M operands are 32-byte pieces of its row, loaded
// straight into registers two steps ahead (two sets used alternately; no wave
// reads another's rows, so M needs no LDS), and S_J, the only thing the waves
// exchange, sits in LDS by columns (two buffers, one barrier a step).  A step is
// bound by the fp32 MFMA rate of its CU (D^2 x 16 products, 1 us): 31 steps at D =
// 128, H 8 take 75 us with M staged in LDS by four waves, 62 in this form.
template <int D>
__global__ void __launch_bounds__(4 * D) k_gdn_scan(GdnArgs a) {
    constexpr int NJ = D / 16, LS = D + 4;
    __shared__ __attribute__((aligned(16))) float sS[2][16 * LS];  // [column][row]
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q4 = lane >> 4, n16 = lane & 15;
    int bh, col0;
    if (!scan_item<D>(a, bh, col0)) return;
    const int64_t SS = (int64_t)D * D;
    const int nJ = a.n_super, last = a.scan_out ? nJ : nJ - 1;  // steps taken
    const float *wsM = a.wsM + (int64_t)bh * a.n_prep * SS, *wsN = a.wsN + (int64_t)bh * a.n_prep * SS;
    float *wsS = a.wsS + (int64_t)bh * nJ * SS;
    // the wave's rows 16w + 4 q4 + r of the state, column col0 + n16 (byte offsets)
    const uint32_t so = (uint32_t)(((16 * w + 4 * q4) * D + col0 + n16) * 4);
    const uint32_t mo = (uint32_t)(((16 * w + n16) * D + 8 * q4) * 4);
    auto get = [&](const float *src) {
        const rsrc_t rs = buf_rsrc(src, (uint32_t)(SS * 4));
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = buf_ld<float>(rs, so, r * D * 4);
        return x;
    };
    auto put = [&](float *dst, const f32x4 &x) {
        const rsrc_t rs = buf_rsrc(dst, (uint32_t)(SS * 4));
#pragma unroll
        for (int r = 0; r < 4; ++r) buf_st(rs, so, r * D * 4, x[r]);
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (a.S_in) acc = get(a.S_in + bh * SS);
    f32x4 mA[NJ], mB[NJ], nA = acc, nB = acc;
    auto fetch = [&](f32x4 (&mr)[NJ], f32x4 &nr, int J) {
        const rsrc_t rs = buf_rsrc(wsM + (int64_t)J * SS, (uint32_t)(SS * 4));
#pragma unroll
        for (int j = 0; j < NJ; ++j) mr[j] = buf_ld<f32x4>(rs, mo, 128 * (j >> 1) + 16 * (j & 1));
        nr = get(wsN + (int64_t)J * SS);
    };
    // step J: store S_J; unless J is the last, S_{J+1} = M_J S_J + N_J from
    // (mr, nr), which then take the maps of J + 2; false after the last store
    auto step = [&](int J, f32x4 (&mr)[NJ], f32x4 &nr) {
        if (J < nJ) put(wsS + (int64_t)J * SS, acc);
        if (J == last) return false;
        float *const s = sS[J & 1];
        *reinterpret_cast<f32x4 *>(&s[n16 * LS + 16 * w + 4 * q4]) = acc;
        __syncthreads();
        acc = nr;
        f32x4 acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const f32x4 b = *reinterpret_cast<const f32x4 *>(&s[n16 * LS + 32 * (j >> 1) + 8 * q4 + 4 * (j & 1)]);
#pragma unroll
            for (int u = 0; u < 4; u += 2) {
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(mr[j][u], b[u], acc, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(mr[j][u + 1], b[u + 1], acc2, 0, 0, 0);
            }
        }
        acc += acc2;
        if (J + 2 < last) fetch(mr, nr, J + 2);
        return true;
    };
    if (last > 0) fetch(mA, nA, 0);
    if (last > 1) fetch(mB, nB, 1);
    for (int J = 0;; J += 2)
        if (!step(J, mA, nA) || !step(J + 1, mB, nB)) break;
    if (a.scan_out) put(a.S_out + bh * SS, acc);  // the state after the last superchunk
}


// ------------------------------------------------------------------ backward
//
// Per chunk, with S the state entering it, dS' the gradient of the state leaving
// it and the forward quantities above (b, gamma, Gamma, A, W, Ubar, U, P):
//   dU  = diag(e^{b_C - b}) K dS' + P^T dO
//   dS  = gamma_C dS' + Q^T diag(gamma) dO - W^T dU          (the state gradient entering)
//   dq  = diag(gamma) dO S^T + (dO U^T o Gamma) K
//   dk  = diag(e^{b_C - b}) U dS'^T + (dO U^T o Gamma)^T Q + diag(beta gamma) G_W + Ah K + Ah^T K
//   dv  = diag(beta) G_U,   [G_W | G_U] = (I + A)^{-T} [-dU S^T | dU]
//   dA  = -(G_W W^T + G_U Ubar^T) on s < t,   Ah = dA o beta_t e^{b_t - b_s}
//   dbeta_t = gamma_t <G_W_t, k_t> + <G_U_t, v_t> + sum_s dA[t][s] e^{b_t - b_s} k_t.k_s
// and the log-decay gradient collects, per token, every term through b_t
// (gamma_t, Gamma, A, e^{b_C - b_t}, gamma_C), summed in reverse over the chunk.
// dS runs backwards over the chunks; it is the chunk map's transpose, so a
// superchunk maps dS_end to dS_start = M_J^T dS_end + E_J, with M_J the forward
// prep's and E_J the walk from dS_end = 0.
//   k_gdn_dwalk<true>:  E_J for J >= 1;
//   k_gdn_dscan:        dS_end(J) for every J (M_{J+1}^T, fp32, in reverse);
//   k_gdn_dwalk<false>: from dS_end(J), writes dS' of every chunk and dS_in;
//   k_gdn_dchunk:       the parameter gradients of every chunk, all chunks in
//                       parallel, from the stored S and dS' (bf16 hi/lo pairs, fp32 sums).

// The backward's state-gradient walk, its waves, columns and tiles as the forward
// walks'.  Per chunk, each wave on its own columns:
//   dU = e^{b_C - b} o (K dS') + P^T dO,   G_U = T^T dU,   dv = beta o G_U,
//   dS = gamma_C dS' + Q^T (gamma o dO) - K^T (beta gamma o G_U)
// (W^T dU = K^T diag(beta gamma) T^T dU, so W is not formed).  dv leaves through
// an MFMA with the identity that turns its rounded values around, so a lane
// stores consecutive channels of a token.
template <typename T, int D, bool PREP>
__global__ void __launch_bounds__(256, 2) k_gdn_dwalk(GdnArgs a) {
    constexpr bool TPRE = D == 128;
    constexpr int NT = 256, NK = D / 16, NCT = GdnCols<D>::NCT;
    constexpr int LDN = D + pad<T>(), SWX = swx<T, D>(), LDA = C + 4;
    __shared__ __attribute__((aligned(16))) T sQ[C * LDN];      // swizzled
    __shared__ __attribute__((aligned(16))) T sK[C * LDN];      // swizzled
    __shared__ __attribute__((aligned(16))) T sO[C * LDN];      // dO, swizzled
    __shared__ __attribute__((aligned(16))) short sT[2 * TRI];  // T, hi then lo
    __shared__ __attribute__((aligned(16))) T sP[2 * TRI];      // P^T[s][t] = e^{b_t-b_s} k_s.q_t (s <= t), hi then lo
    __shared__ __attribute__((aligned(16))) float sA[TPRE ? 4 : C * LDA];
    __shared__ __attribute__((aligned(16))) float sb[C], sq[C], se[C], sbeta[C];

    const int tid = threadIdx.x, lane = tid & 63, q4 = lane >> 4, n16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const GdnCols<D> cl{16 * NCT * w, n16};
    const int nJ = PREP ? a.n_super - 1 : a.n_super;
    const int item = blockIdx.x, bh = item / nJ, J = (PREP ? 1 : 0) + item % nJ;
    const int bb = bh / a.H, hh = bh % a.H;
    const int64_t tok0 = (int64_t)J * a.ts;
    const int64_t xo = bb * a.sx_b + hh * a.sx_h + tok0 * a.sx_l;
    const T *Q = (const T *)a.q + xo;
    const T *K = (const T *)a.k + xo;
    const T *DO = (const T *)a.dO + xo;
    const T *TW = TPRE ? (const T *)a.tw + xo : nullptr;
    T *DV = (T *)a.dv + xo;
    const int64_t go = bb * a.sg_b + hh * a.sg_h + tok0 * a.sg_l;
    const float *gp = a.g + go;
    const float *bp = a.beta + go;
    const int64_t SS = (int64_t)D * D;
    const int nch = (int)((a.L - tok0 < a.ts ? a.L - tok0 : a.ts) / C);
    const LaneOff swo = swz_off<T, LDN, SWX>(lane), tro8 = tr_off8<T, LDN, SWX>(lane);
    const LaneOff tro = NCT == 2 ? tro8 : tr_off<T, LDN, SWX>(lane);  // this wave's own columns
    // rows of the accumulators and of the fragments that build them: see the forward walk
    auto prow = [&](int i, int r) { return 32 * (i >> 1) + 8 * q4 + 4 * (i & 1) + r; };
    const int ar = 8 * (n16 >> 2) + (n16 & 3);
    auto roff = [](int i) { return 32 * (i >> 1) + 4 * (i & 1); };
    const LaneOff ko = {ar * LDN + 8 * q4 + ((n16 >> 2) & 1) * SWX, ar * LDN + 8 * q4 - ((n16 >> 2) & 1) * SWX};

    const int ta = tri_pos<0>(ar, 8 * q4);
    const int tt8 = tri_pos<0>(8 * q4 + (n16 >> 2), 8 * (n16 & 3));  // T's transposing reads

    // dS[m][i][r] = dS[prow(i, r)][col(m)]: from dS_end(J) (dS_out for one superchunk), or 0 (prep)
    const StateIO<D> sio(cl, q4);
    f32x4 dS[NCT][NK];
#pragma unroll
    for (int m = 0; m < NCT; ++m)
#pragma unroll
        for (int i = 0; i < NK; ++i) dS[m][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (!PREP) {
        const float *src = a.n_super == 1 ? (a.dS_out ? a.dS_out + bh * SS : nullptr)
                                          : a.wsDe + ((int64_t)bh * a.n_super + J) * SS;
        if (src) sio.load(dS, src);
    }

    using TT = Tile<T, D, NT>;
    TT t1, t2, t3;
    TriTile<T> t4;
    float gl = 0.f, bl = 0.f;  // wave 3's: a load of a chunk's gates touches 64 cache lines
    const int64_t cstep = (int64_t)C * a.sx_l;
    const uint32_t cspan = chunk_span<T, D>(a.sx_l), gspan = (uint32_t)(((C - 1) * a.sg_l + 1) * 4);
    uint32_t toff[TT::RPT];
    TT::offsets(toff, a.sx_l, tid);
    const uint32_t goff = (uint32_t)(lane * a.sg_l * 4);
    const uint32_t tstep = (uint32_t)(16 * a.sx_l * (int64_t)sizeof(T));
    const int t4base = TriTile<T>::base(tid);
    const uint32_t t4off = (uint32_t)(((tid >> 4) * a.sx_l + 8 * (tid & 15)) * (int64_t)sizeof(T));
    const uint32_t voff = (uint32_t)((n16 * a.sx_l + cl.c0 + 4 * NCT * q4) * (int64_t)sizeof(T));
    const uint32_t coff = (uint32_t)(cl.col(0) * D + 8 * q4) * 2;  // chunk state pairs
    auto issue = [&](int c) {
        const int64_t nx = c * cstep;
        t1.load_buf(buf_rsrc(Q + nx, cspan), toff, 0);
        t2.load_buf(buf_rsrc(K + nx, cspan), toff, 0);
        if (w == 3) {
            gl = buf_ld<float>(buf_rsrc(gp + (int64_t)c * C * a.sg_l, gspan), goff, 0);
            bl = buf_ld<float>(buf_rsrc(bp + (int64_t)c * C * a.sg_l, gspan), goff, 0);
        }
        if constexpr (TPRE) t4.load(buf_rsrc(TW + nx, cspan), t4off, tstep, tid);
        t3.load_buf(buf_rsrc(DO + nx, cspan), toff, 0);
    };
    if (nch > 0) issue(nch - 1);

    const unsigned par = pair_parity(a.n_cu);
    for (int c = nch - 1; c >= 0; --c) {
        pair_turn(par);
        __syncthreads();  // the previous chunk is done with every LDS tile
        t1.store_swz(sQ, LDN, tid, SWX);
        t2.store_swz(sK, LDN, tid, SWX);
        t3.store_swz(sO, LDN, tid, SWX);
        if constexpr (TPRE) t4.store(sT, t4base, tid);
        if (w == 3) {
            const float b2 = wave_scan_dpp(gl * LOG2E);
            const float b63 = lane_value(b2, 63);
            sb[lane] = b2;
            sq[lane] = fexp2(b2);
            se[lane] = fexp2(b63 - b2);
            sbeta[lane] = bl;
        }
        __syncthreads();

        // P^T on the causal tiles: rows t of the accumulator, 4 of one row s of P^T
        for (int i = w; i < 10; i += 4) {
            int tt, st;
            tri_tile(i, tt, st);
            f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < D / 32; ++ks)
                mma(p, ldfrag_swz<T, LDN, SWX>(sQ, swo, 16 * tt, 32 * ks), ldfrag_swz<T, LDN, SWX>(sK, swo, 16 * st, 32 * ks));
            const int s = 16 * st + n16;
            const float bs = sb[s];
            const f32x4 bt = *reinterpret_cast<const f32x4 *>(&sb[16 * tt + 4 * q4]);
            float v4[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v4[r] = s <= 16 * tt + 4 * q4 + r ? p[r] * fexp2(bt[r] - bs) : 0.f;
            const int o = tri_pos<0>(s, 16 * tt + 4 * q4);
            st4_split<T, true>(&sP[o], &sP[TRI + o], v4);
        }
        if (tid < 128) {  // the zero blocks (1,0) and (3,2) of the diagonal quadrants
            const int b = tid >> 6, o = tri_pos<0>(32 * b + 16 + ((tid >> 2) & 15), 32 * b + 4 * (tid & 3));
            *reinterpret_cast<s4v *>(&sP[o]) = s4v{0, 0, 0, 0};
            *reinterpret_cast<s4v *>(&sP[TRI + o]) = s4v{0, 0, 0, 0};
        }
        if constexpr (!TPRE) {
            gdn_a_scores<T, D, LDN, SWX>(w, lane, sK, sb, sbeta, sA);
            __syncthreads();
            gdn_tinv_hl(tid, sA, sT, sT + TRI);
        }

        // dU[t][v] = e^{b_C - b_t} sum_k K[t][k] dS[k][v] + sum_{t' >= t} P^T[t][t'] dO[t'][v]
        // (rows t = prow(tt, r))
        // dS' of chunk c, the gradient of the state leaving it, is stored on the way
        const rsrc_t rc = buf_rsrc(PREP ? nullptr : a.wsDc + ((int64_t)bh * (a.L / C) + tok0 / C + c) * SS, D * D * 4);
        f32x4 dU[NCT][4];
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) dU[m][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
            frag_t<T> fh[NCT], fl[NCT];
#pragma unroll
            for (int m = 0; m < NCT; ++m) {
                split_acc<T, true>(dS[m][2 * ks], dS[m][2 * ks + 1], fh[m], fl[m]);
                if constexpr (!PREP) put_state_pair<T, D>(rc, coff, m, ks, fh[m], fl[m]);
            }
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const frag_t<T> kf = *reinterpret_cast<const frag_t<T> *>(
                    &sK[(((32 * ks) & SWX) ? ko.hi : ko.lo) + roff(tt) * LDN + 32 * ks]);
#pragma unroll
                for (int m = 0; m < NCT; ++m) {
                    mma(dU[m][tt], kf, fh[m]);
                    mma(dU[m][tt], kf, fl[m]);
                }
            }
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const f32x4 ev = *reinterpret_cast<const f32x4 *>(&se[prow(tt, 0)]);
#pragma unroll
            for (int m = 0; m < NCT; ++m) dU[m][tt] *= ev;
        }
        __syncthreads();  // P^T is complete
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            frag_t<T> of[NCT];
#pragma unroll
            for (int m = 0; m < NCT; ++m) of[m] = ldfragTR<T, LDN, SWX>(sO, tro, 32 * ks, cl.base(m));
#pragma unroll
            for (int tt = 0; tt < 2 * ks + 2; ++tt) {
                const frag_t<T> ph = *reinterpret_cast<const frag_t<T> *>(&sP[ta + tri_a(tt, ks)]);
                const frag_t<T> pl = *reinterpret_cast<const frag_t<T> *>(&sP[ta + TRI + tri_a(tt, ks)]);
#pragma unroll
                for (int m = 0; m < NCT; ++m) {
                    mma(dU[m][tt], ph, of[m]);
                    mma(dU[m][tt], pl, of[m]);
                }
            }
        }
        // G_U[s][v] = sum_{t >= s} T[t][s] dU[t][v] (rows s = prow(tt, r))
        f32x4 G[NCT][4];
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) G[m][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // rows s = ar + roff(tt), contraction t = 32 ks + 8 q4 + j (the swizzle ignores row bit 2)
        auto t_tr = [&](const short *M, int ks, int tt) {
            typedef short s8 __attribute__((ext_vector_type(8)));
            const short *p = M + tt8 + (ks + (tt >> 1)) * 1024 + 4 * (tt & 1);
            const s4v x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)p);
            const s4v x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)(p + 4 * 32));
            const s8 v = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(frag_t<T>, v);
        };
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            frag_t<T> xh[NCT], xl[NCT];
#pragma unroll
            for (int m = 0; m < NCT; ++m) split_acc<T, true>(dU[m][2 * ks], dU[m][2 * ks + 1], xh[m], xl[m]);
#pragma unroll
            for (int tt = 0; tt < 2 * ks + 2; ++tt) {
                const frag_t<T> th = t_tr(sT, ks, tt), tl = t_tr(sT + TRI, ks, tt);
#pragma unroll
                for (int m = 0; m < NCT; ++m) {
                    mma(G[m][tt], th, xh[m]);
                    mma(G[m][tt], th, xl[m]);
                    mma(G[m][tt], tl, xh[m]);
                }
            }
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const f32x4 be = *reinterpret_cast<const f32x4 *>(&sbeta[prow(tt, 0)]);
#pragma unroll
            for (int m = 0; m < NCT; ++m) G[m][tt] *= be;
        }
        if constexpr (!PREP) {  // dv[s][v], turned to rows v, columns s = 16 tt + n16
            const rsrc_t rv = buf_rsrc(DV + c * cstep, cspan);
            frag_t<T> eye[2];  // column 16 tt + n16 of tile tt against its own 32 tokens
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 8; ++j) eye[h][j] = (T)(q4 == 2 * h + (n16 >> 3) && j == (n16 & 7) ? 1.f : 0.f);
#pragma unroll
            for (int ks = 0; ks < C / 32; ++ks) {
                frag_t<T> vf[NCT];
#pragma unroll
                for (int m = 0; m < NCT; ++m) vf[m] = frag_from_acc<T>(G[m][2 * ks], G[m][2 * ks + 1]);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    f32x4 o[NCT];
#pragma unroll
                    for (int m = 0; m < NCT; ++m) {
                        o[m] = f32x4{0.f, 0.f, 0.f, 0.f};
                        mma(o[m], vf[m], eye[h]);
                    }
                    if constexpr (NCT == 2) {
                        typedef T v8 __attribute__((ext_vector_type(8)));
                        v8 x = {};
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            x[r] = cvt<T>(o[0][r]);
                            x[4 + r] = cvt<T>(o[1][r]);
                        }
                        buf_st(rv, voff, (2 * ks + h) * tstep, x);
                    } else {
                        st4_buf<T>(rv, voff, (2 * ks + h) * tstep, o[0]);
                    }
                }
            }
        }

        if (c > 0) issue(c - 1);

        // dS = gamma_C dS + Q^T (gamma o dO) - K^T (beta gamma o G_U)
        const float gam = sq[C - 1];
#pragma unroll
        for (int m = 0; m < NCT; ++m)
#pragma unroll
            for (int i = 0; i < NK; ++i) dS[m][i] *= gam;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const f32x4 gq = *reinterpret_cast<const f32x4 *>(&sq[prow(tt, 0)]);
#pragma unroll
            for (int m = 0; m < NCT; ++m) G[m][tt] *= -gq;
        }
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            const f32x4 g0 = *reinterpret_cast<const f32x4 *>(&sq[32 * ks + 8 * q4]);
            const f32x4 g1 = *reinterpret_cast<const f32x4 *>(&sq[32 * ks + 8 * q4 + 4]);
            const float gt[8] = {g0[0], g0[1], g0[2], g0[3], g1[0], g1[1], g1[2], g1[3]};
            frag_t<T> gh[NCT], glo[NCT], uh[NCT], ul[NCT];
#pragma unroll
            for (int m = 0; m < NCT; ++m) {
                split_scaled<T, true>(ldfragTR<T, LDN, SWX>(sO, tro, 32 * ks, cl.base(m)), gt, gh[m], glo[m]);
                split_acc<T, true>(G[m][2 * ks], G[m][2 * ks + 1], uh[m], ul[m]);
            }
#pragma unroll
            for (int i = 0; i < NK; ++i) {
                const frag_t<T> qf = ldfragTR<T, LDN, SWX>(sQ, tro8, 32 * ks, roff(i));
                const frag_t<T> kf = ldfragTR<T, LDN, SWX>(sK, tro8, 32 * ks, roff(i));
#pragma unroll
                for (int m = 0; m < NCT; ++m) {
                    mma2b<T, true>(dS[m][i], qf, gh[m], glo[m]);
                    mma2b<T, true>(dS[m][i], kf, uh[m], ul[m]);
                }
            }
        }
    }
    float *dst = PREP ? a.wsE + ((int64_t)bh * (a.n_super - 1) + J - 1) * SS : (J == 0 ? a.dS_in + bh * SS : nullptr);
    if (dst) sio.store(dS, dst);
}

// dS_end(n-1) = dS_out (or 0); dS_end(J-1) = M_J^T dS_end(J) + E_J, written to
// wsDe for every J.  Same shape of work as k_gdn_scan, with M_J read transposed:
// slot m of the contraction is k = 4 m + q4, so a lane loads one column of M_J, the
// lanes of a row 64 consecutive bytes.
template <int D>
__global__ void __launch_bounds__(4 * D) k_gdn_dscan(GdnArgs a) {
    constexpr int NM = D / 4, LS = D + 4;
    __shared__ __attribute__((aligned(16))) float sS[2][16 * LS];  // [column][slot]: slot NM q4 + m is row 4 m + q4
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, q4 = lane >> 4, n16 = lane & 15;
    int bh, col0;
    if (!scan_item<D>(a, bh, col0)) return;
    const int64_t SS = (int64_t)D * D;
    const int nJ = a.n_super;
    float *wsDe = a.wsDe + (int64_t)bh * nJ * SS;
    const float *wsM = a.wsM + (int64_t)bh * a.n_prep * SS, *wsE = a.wsE + (int64_t)bh * (nJ - 1) * SS;
    const uint32_t so = (uint32_t)(((16 * w + 4 * q4) * D + col0 + n16) * 4);
    const uint32_t mo = (uint32_t)((q4 * D + 16 * w + n16) * 4);
    auto get = [&](const float *src) {
        const rsrc_t rs = buf_rsrc(src, (uint32_t)(SS * 4));
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = buf_ld<float>(rs, so, r * D * 4);
        return x;
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (a.dS_out) acc = get(a.dS_out + bh * SS);
    float mA[NM], mB[NM];
    f32x4 nA = acc, nB = acc;
    auto fetch = [&](float (&mr)[NM], f32x4 &nr, int J) {
        const rsrc_t rs = buf_rsrc(wsM + (int64_t)J * SS, (uint32_t)(SS * 4));
#pragma unroll
        for (int m = 0; m < NM; ++m) mr[m] = buf_ld<float>(rs, mo, 4 * m * D * 4);
        nr = get(wsE + (int64_t)(J - 1) * SS);
    };
    // step J: store dS_end(J); unless J = 0, dS_end(J-1) = M_J^T dS_end(J) +
    // E_{J-1} from (mr, nr), which then take the maps of J - 2; false after J = 0
    auto step = [&](int J, float (&mr)[NM], f32x4 &nr) {
        const rsrc_t rs = buf_rsrc(wsDe + (int64_t)J * SS, (uint32_t)(SS * 4));
        float *const s = sS[J & 1];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            buf_st(rs, so, r * D * 4, acc[r]);
            s[n16 * LS + NM * r + 4 * w + q4] = acc[r];  // row 16w + 4 q4 + r
        }
        if (J == 0) return false;
        __syncthreads();
        acc = nr;
        f32x4 acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < NM; m += 4) {
            const f32x4 b = *reinterpret_cast<const f32x4 *>(&s[n16 * LS + NM * q4 + m]);
#pragma unroll
            for (int u = 0; u < 4; u += 2) {
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(mr[m + u], b[u], acc, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(mr[m + u + 1], b[u + 1], acc2, 0, 0, 0);
            }
        }
        acc += acc2;
        if (J - 2 >= 1) fetch(mr, nr, J - 2);
        return true;
    };
    if (nJ > 1) fetch(mA, nA, nJ - 1);
    if (nJ > 2) fetch(mB, nB, nJ - 2);
    for (int J = nJ - 1;; J -= 2)
        if (!step(J, mA, nA) || !step(J - 1, mB, nB)) break;
}

// Parameter gradients of one chunk per item (b, h, chunk), items in a grid-stride
// loop, one workgroup of D / 16 waves per CU.  S is the state entering the chunk
// and dS' the gradient of the state leaving it, both stored per chunk by the walks
// as transposed hi/lo pairs (put_state_pair).  Three identities keep W, Ubar and a
// second inverse out of the kernel:
//   U = T diag(beta) (V - diag(gamma) K S),   G_U = T^T dU,
//   G_W = T^T (-dU S^T) = -G_U S^T,   dA = -(G_W W^T + G_U Ubar^T) = -G_U U^T.
// Wave w owns the 16 channels [16w, 16w + 16) throughout:
//   1. of v: Y = K S, dU = e o (K dS') + P^T dO on its own columns of S and dS',
//      which go from memory straight into its registers; U^T and G_U^T (rows v)
//      leave their accumulators as four consecutive channels of a token, into LDS
//      as hi/lo pairs;
//   2. of k: dQ_S^T = S dO^T, G_W^T = -S G_U^T, dK_S^T = dS' U^T on its own rows
//      of S and dS', handed on through LDS 32 columns at a time (read again from
//      memory, both missed L2 often enough to cost a third more traffic);
//   3. the causal 16 x 16 tiles of dA and dP = dO U^T, shared out over the waves,
//      become E1 = dP o Gamma and E2 = Ah + Ah^T (Ah = dA o beta Gamma) in LDS;
//   4. dq = gamma dQ_S + E1 K,  dk = e dK_S + E1^T Q + beta gamma G_W + E2 K, turned
//      into whole rows through LDS.
// Thirteen barriers per item.  dbeta and the log-decay gradient come from row and
// column sums in a fixed order (no atomics).  q, k, v, dO enter the products
// exactly (bf16); the computed fp32 operands (S, dS', T, P, X, U, dU, G_U, E1, E2)
// as hi/lo bf16 pairs (three products, lo x lo dropped; kept in <dS', S>, which all
// of dg is at weak decay: without it dg was 7.5e-6 off at g = -e^-8, with it 7.0e-6).
// The next item's q, k, T, S and dS' wait in registers from step 2 on and its v, dO
// are copied into LDS during step 4.
// D = 128, 65536 tokens of 40 heads: 7.6 ms with S and dS' staged through LDS in
// blocks of 32 channels by 16 waves (T formed again, spills), 3.0 ms so (10.9 GB
// moved, 9.9 of them needed; 2.1 ms at the rate of a copy).
template <typename T, int D>
__global__ void __launch_bounds__(4 * D, 1) k_gdn_dchunk(GdnArgs a) {
    constexpr int NW = D / 16, NT = 4 * D, KS = D / 32, BPR = D / 8;
    constexpr bool TPRE = D == 128;
    constexpr int XT = C * D;          // elements of a chunk tile
    // tiles in DmaTile's layout; G_U's hi half takes v's place (a lane overwrites
    // the values that it alone has read)
    __shared__ __attribute__((aligned(16))) T sQ[XT], sK[XT], sO[XT], sUh[XT], sUl[XT], sGh[XT], sGl[XT];
    // T then E1 (tri, 12 KB), P^T then part of E2 (full C x C pair); between the two,
    // four planes of 32 x D
    constexpr int RN = 2 * TRI + 2 * C * C > 128 * D ? 2 * TRI + 2 * C * C : 128 * D;
    __shared__ __attribute__((aligned(16))) short sR[RN];
    __shared__ __attribute__((aligned(16))) float sb[C], sg[C], se[C], sbe[C];
    __shared__ float sGv[NW][C];                                   // per wave: G_U.v
    __shared__ float sRX[4][C], sXr[2][4][C], sXc[2][4][C];        // per tile column / row: see the sums below
    __shared__ float sWav[NW];
    __shared__ __attribute__((aligned(16))) float sA[TPRE ? 4 : C * (C + 4)];
    T *const sV = sGh;
    // per wave: G_W.k, dK_S.k, gamma q.dQ_S, once G_U is no longer read
    typedef float row_t[C];
    row_t *const sZ = reinterpret_cast<row_t *>(sGl), *const sW = sZ + NW, *const sY = sW + NW;
    static_assert(3 * NW * C * 4 <= XT * (int)sizeof(T), "the sums fit G_U's lo tile");
    short *const sT = sR;
    T *const sP = reinterpret_cast<T *>(sR + 2 * TRI);
    T *const sE1 = reinterpret_cast<T *>(sR), *const sE2 = reinterpret_cast<T *>(sR + 2 * TRI);

    const int tid = threadIdx.x;
    int lane = tid & 63, q4 = lane >> 4, n16 = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t SS = (int64_t)D * D;
    // (the chunk states of 2^31 items would not fit any memory)
    const uint32_t nc = (uint32_t)(a.L / C), items = (uint32_t)(a.B * a.H) * nc;

    // --- positions (see DmaTile for the swizzle)
    auto xpos = [](int r, int c) { return r * D + (((c >> 3) ^ (r & 7) ^ (((r >> 3) & 1) << 2)) << 3) + (c & 7); };
    auto epos = [](int r, int c) { return r * C + (((c >> 3) ^ (r & 7)) << 3) + (c & 7); };  // E2
    auto roff = [](int i) { return 32 * (i >> 1) + 4 * (i & 1); };
    auto prow = [&](int i, int r) { return 32 * (i >> 1) + 8 * q4 + 4 * (i & 1) + r; };
    // The lane's positions, and the lane index itself, opaque to the compiler: it
    // would otherwise form every LDS address ahead of the item loop and keep them
    // all (180 registers spilled).
    int rb[2], kb[2], tb[2], ub[2], eb[2], ar, own, trb, tra, xb;
    auto positions = [&]() {
        asm volatile("" : "+v"(lane));
        q4 = lane >> 4;
        n16 = lane & 15;
        DmaTile<T, D, NW>::row_base(lane, rb);  // rows 16 tt + n16: rb[ks & 1] + 16 tt D + 64 (ks >> 1)
        ar = 8 * (n16 >> 2) + (n16 & 3);        // rows ar + roff(tt): kb[(ks ^ tt) & 1] + roff(tt) D + 64 (ks >> 1)
        kb[0] = ar * D + 8 * ((q4 ^ (n16 & 3)) | (4 * ((n16 >> 2) & 1)));
        kb[1] = ar * D + 8 * ((q4 ^ (n16 & 3)) | (4 * (1 ^ ((n16 >> 2) & 1))));
        const int r0 = 8 * q4 + (n16 >> 2), ch = 4 * (n16 & 3);
        tb[0] = xpos(r0, 16 * w + ch);  // transposing reads of the wave's own channels: tb[0] + 32 ks D, tb[1] four rows on
        tb[1] = xpos(r0 + 4, 16 * w + ch);
        ub[0] = tri_pos<0>(r0, ch);     // ... of a triangular tile's columns 16 i ..: ub[i & 1] + (ks + i / 2) 1024
        ub[1] = tri_pos<0>(r0, 16 + ch);
        trb = tri_pos<0>(n16, 8 * q4);  // its rows 16 tt + n16: trb + tri_b; rows ar + roff(tt): tra + tri_a
        tra = tri_pos<0>(ar, 8 * q4);
        eb[0] = epos(n16, 8 * q4);      // E2: rows 16 tt + n16, columns 32 ks + 8 q4 ..: eb[ks] + 16 tt C
        eb[1] = epos(n16, 32 + 8 * q4);
        own = 16 * w + 4 * q4;          // accumulator rows: channels own + r
        xb = xpos(n16, own);            // token 16 tt + n16, channels own ..: xb + 16 tt D
    };
    positions();
    auto rd = [](const T *M, int p) { return *reinterpret_cast<const frag_t<T> *>(M + p); };
    auto rows = [&](const T *M, int tt, int ks) { return rd(M, rb[ks & 1] + 16 * tt * D + 64 * (ks >> 1)); };
    auto tr2 = [](const void *p0, const void *p1) {
        typedef short s8 __attribute__((ext_vector_type(8)));
        const s4v x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)p0);
        const s4v x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4v *)p1);
        const s8 v = __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(frag_t<T>, v);
    };
    auto cols = [&](const T *M, int ks) { return tr2(M + tb[0] + 32 * ks * D, M + tb[1] + 32 * ks * D); };
    auto tri_tr = [&](const short *M, int ks, int i) {  // rows 16 i + n16 of M^T, contraction 32 ks + 8 q4 + j
        const short *p = M + ub[i & 1] + (ks + (i >> 1)) * 1024;
        return tr2(p, p + 4 * 32);
    };
    auto tri_rows = [&](const short *M, int tt, int ks) {  // rows 16 tt + n16, columns 32 ks + 8 q4 ..
        return rd(reinterpret_cast<const T *>(M), trb + tri_b(tt, ks));
    };
    auto mma3 = [](f32x4 &c, const frag_t<T> &ah, const frag_t<T> &al, const frag_t<T> &bh, const frag_t<T> &bl) {
        mma(c, ah, bh);
        mma(c, ah, bl);
        mma(c, al, bh);
    };
    auto sum16 = [](float v) {  // over the 16 lanes of a row, in every lane
        v += dpp_or0<0x128>(v);
        v += dpp_or0<0x124>(v);
        v += dpp_or0<0x122>(v);
        v += dpp_or0<0x121>(v);
        return v;
    };
    // four values of four consecutive channels / columns as a hi/lo pair
    auto put4 = [](T *h, T *l, int p, const f32x4 &x) {
        const float v[4] = {x[0], x[1], x[2], x[3]};
        st4_split<T, true>(h + p, l + p, v);
    };
    const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
    // --- loads of an item
    typedef s4v2 blk;
    const DmaTile<T, D, NW> dma(lane, a.sx_l);
    const uint32_t rowb = (uint32_t)(a.sx_l * (int64_t)sizeof(T)), span = chunk_span<T, D>(a.sx_l);
    const uint32_t xoff = (uint32_t)((tid / BPR) * (uint64_t)rowb + 16 * (tid % BPR));  // block tid of a tile
    const int sp = xpos(tid / BPR, 8 * (tid % BPR));
    const uint32_t toff = (uint32_t)((tid >> 4) * (uint64_t)rowb + 16 * (tid & 15));
    blk pq[2], pk[2], pt[2];
    float gl = 0.f, bl = 0.f;
    frag_t<T> s1h[KS], s1l[KS], d1h[KS], d1l[KS];  // S, dS' of the wave's own v: [own v][32 ks + 8 q4 ..]
    // offsets of an item's tokens and gates
    auto locate = [&](uint32_t it, int64_t &xo, int64_t &go) {
        const uint32_t bh = it / nc, ch = it - bh * nc, b = bh / (uint32_t)a.H, h = bh - b * (uint32_t)a.H;
        xo = b * a.sx_b + h * a.sx_h + (int64_t)(ch * C) * a.sx_l;
        go = b * a.sg_b + h * a.sg_h + (int64_t)(ch * C) * a.sg_l;
    };
    constexpr uint32_t RS = NT / BPR, RT = NT / 16;  // rows per round of blocks: tiles, T
    auto load_regs = [&](int64_t xo, int64_t go) {
        const rsrc_t rq = buf_rsrc((const T *)a.q + xo, span), rk = buf_rsrc((const T *)a.k + xo, span);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            pq[i] = buf_ld<blk>(rq, xoff, i * RS * rowb);
            pk[i] = buf_ld<blk>(rk, xoff, i * RS * rowb);
        }
        if constexpr (TPRE) {
            const rsrc_t rt = buf_rsrc((const T *)a.tw + xo, span);
            if ((tid & 7) < 4) pt[0] = buf_ld<blk>(rt, toff, 0);
            pt[1] = buf_ld<blk>(rt, toff, RT * rowb);
        }
        if (w == 0) {  // one cache line per token: a load costs 64 of them, so one wave does it
            const uint32_t gspan = (uint32_t)(((C - 1) * a.sg_l + 1) * 4), goff = (uint32_t)(lane * a.sg_l * 4);
            gl = buf_ld<float>(buf_rsrc(a.g + go, gspan), goff, 0);
            bl = buf_ld<float>(buf_rsrc(a.beta + go, gspan), goff, 0);
        }
    };
    auto load_vo = [&](int64_t xo) {
        dma.issue(buf_rsrc((const T *)a.v + xo, span), sV, w, rowb);
        dma.issue(buf_rsrc((const T *)a.dO + xo, span), sO, w, rowb);
    };
    auto load_s1 = [&](uint32_t it) {
        const rsrc_t rs = buf_rsrc(a.wsSc + (int64_t)it * SS, (uint32_t)(SS * 4)), rd = buf_rsrc(a.wsDc + (int64_t)it * SS, (uint32_t)(SS * 4));
        const uint32_t o = (uint32_t)(((16 * w + n16) * D + 8 * q4) * 2);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            s1h[ks] = buf_ld<frag_t<T>>(rs, o, 64 * ks);
            s1l[ks] = buf_ld<frag_t<T>>(rs, o, 64 * ks + D * D * 2);
            d1h[ks] = buf_ld<frag_t<T>>(rd, o, 64 * ks);
            d1l[ks] = buf_ld<frag_t<T>>(rd, o, 64 * ks + D * D * 2);
        }
    };

    uint32_t it = blockIdx.x;
    if (it >= items) return;
    int64_t xo, go, xn = 0, gn = 0;
    locate(it, xo, go);
    load_regs(xo, go);
    load_vo(xo);
    vm_wait_all();
    load_s1(it);
    for (;; it += gridDim.x, xo = xn, go = gn) {
        const uint32_t nx = it + gridDim.x;  // (below 2^32: see items)
        if (nx < items) locate(nx, xn, gn);
        positions();
        // --- stage
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int p = sp + i * RS * D;  // (RS a multiple of 16: the swizzle repeats)
            *reinterpret_cast<blk *>(sQ + p) = pq[i];
            *reinterpret_cast<blk *>(sK + p) = pk[i];
        }
        if constexpr (TPRE) {
            const int j = tid & 15, c8 = 8 * (j & 7);
            short *const t = sT + (j < 8 ? 0 : TRI);
            if ((tid & 7) < 4) *reinterpret_cast<blk *>(t + tri_pos<0>(tid >> 4, c8)) = pt[0];
            *reinterpret_cast<blk *>(t + tri_pos<0>(32 + (tid >> 4), c8)) = pt[1];
        }
        if (w == 0) {
            const float b2 = wave_scan_dpp(gl * LOG2E);
            const float b63 = lane_value(b2, 63);
            sb[lane] = b2;
            sg[lane] = fexp2(b2);
            se[lane] = fexp2(b63 - b2);
            sbe[lane] = bl;
        }
        __syncthreads();

        // --- P^T on the causal tiles (as in the dS walk)
        for (int i = w; i < 10; i += NW) {
            int tt, st;
            tri_tile(i, tt, st);
            f32x4 p = z4;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) mma(p, rows(sQ, tt, ks), rows(sK, st, ks));
            const int s = 16 * st + n16;
            const float bs = sb[s];
            const f32x4 bt = *reinterpret_cast<const f32x4 *>(&sb[16 * tt + 4 * q4]);
            f32x4 v = z4;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = s <= 16 * tt + 4 * q4 + r ? p[r] * fexp2(bt[r] - bs) : 0.f;
            put4(sP, sP + TRI, tri_pos<0>(s, 16 * tt + 4 * q4), v);
        }
        if (tid < 128) {
            const int b = tid >> 6, o = tri_pos<0>(32 * b + 16 + ((tid >> 2) & 15), 32 * b + 4 * (tid & 3));
            *reinterpret_cast<s4v *>(&sP[o]) = s4v{0, 0, 0, 0};
            *reinterpret_cast<s4v *>(&sP[TRI + o]) = s4v{0, 0, 0, 0};
        }
        if constexpr (!TPRE) {  // T formed here
            for (int i = w; i < 10; i += NW) {
                int tt, st;
                tri_tile(i, tt, st);
                f32x4 p = z4;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) mma(p, rows(sK, st, ks), rows(sK, tt, ks));
                const int t = 16 * tt + n16;
                const float bt = sb[t], be = sbe[t];
                const f32x4 bs = *reinterpret_cast<const f32x4 *>(&sb[16 * st + 4 * q4]);
                f32x4 v = z4;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = 16 * st + 4 * q4 + r < t ? be * p[r] * fexp2(bt - bs[r]) : 0.f;
                *reinterpret_cast<f32x4 *>(&sA[t * (C + 4) + 16 * st + 4 * q4]) = v;
            }
            __syncthreads();
            gdn_tinv_hl(tid, sA, sT, sT + TRI);
        }

        // --- 1. Y = K S, dU = e o (K dS') on the wave's own v (rows t = prow(tt, r))
        f32x4 x[4], du[4], sd4 = z4;  // sd4: (S^T dS')[v][v'], its diagonal sums to <dS', S>, lo x lo included
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) x[tt] = du[tt] = z4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const frag_t<T> sh = s1h[ks], sl = s1l[ks], dh = d1h[ks], dl = d1l[ks];
            mma3(sd4, sh, sl, dh, dl);
            mma(sd4, sl, dl);
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const frag_t<T> kf = rd(sK, kb[(ks ^ tt) & 1] + roff(tt) * D + 64 * (ks >> 1));
                mma(x[tt], kf, sh);
                mma(x[tt], kf, sl);
                mma(du[tt], kf, dh);
                mma(du[tt], kf, dl);
            }
            sched_fence();
        }
        {
            float sd = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) sd += 4 * q4 + r == n16 ? sd4[r] : 0.f;
            sd = wave_sum(sd);
            if (lane == 0) sWav[w] = sd;
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            x[tt] *= -*reinterpret_cast<const f32x4 *>(&sg[prow(tt, 0)]);
            du[tt] *= *reinterpret_cast<const f32x4 *>(&se[prow(tt, 0)]);
        }
        frag_t<T> eye[2];  // as in the forward walk
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 8; ++j) eye[h][j] = (T)(q4 == (n16 >> 2) && j == 4 * h + (n16 & 3) ? 1.f : 0.f);
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {  // X = V - gamma Y
            const frag_t<T> vf = cols(sV, ks);
            mma(x[2 * ks], eye[0], vf);
            mma(x[2 * ks + 1], eye[1], vf);
        }
        sched_fence();
        // U^T[v][t] = sum_s (beta X)^T[v][s] T[t][s]: rows v = own + r, columns t = 16 tt + n16
        f32x4 ut[4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            x[tt] *= *reinterpret_cast<const f32x4 *>(&sbe[prow(tt, 0)]);
            ut[tt] = z4;
        }
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            frag_t<T> xh, xl;
            split_acc<T, true>(x[2 * ks], x[2 * ks + 1], xh, xl);
#pragma unroll
            for (int tt = 2 * ks; tt < 4; ++tt) mma3(ut[tt], xh, xl, tri_rows(sT, tt, ks), tri_rows(sT + TRI, tt, ks));
        }
        __syncthreads();  // P^T is complete
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) put4(sUh, sUl, xb + 16 * tt * D, ut[tt]);
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            const frag_t<T> of = cols(sO, ks);
#pragma unroll
            for (int tt = 0; tt < 2 * ks + 2; ++tt) {
                const int o = tra + tri_a(tt, ks);
                mma(du[tt], rd(sP, o), of);
                mma(du[tt], rd(sP, TRI + o), of);
            }
        }
        sched_fence();
        // G_U^T[v][s] = sum_t dU^T[v][t] T[t][s]; v.G_U per token; G_U over v's place
        f32x4 gt[4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) gt[tt] = z4;
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            frag_t<T> uh, ul;
            split_acc<T, true>(du[2 * ks], du[2 * ks + 1], uh, ul);
#pragma unroll
            for (int tt = 0; tt < 2 * ks + 2; ++tt) mma3(gt[tt], uh, ul, tri_tr(sT, ks, tt), tri_tr(sT + TRI, ks, tt));
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const int p = xb + 16 * tt * D;
            const f32x4 vv = ld4f(sV + p);
            const float gv = sum_rows(gt[tt][0] * vv[0] + gt[tt][1] * vv[1] + gt[tt][2] * vv[2] + gt[tt][3] * vv[3]);
            if (q4 == 0) sGv[w][16 * tt + n16] = gv;
            put4(sGh, sGl, p, gt[tt]);
        }
        __syncthreads();
        positions();
        // --- 2. rows k' = own + r, columns t = 16 tt + n16
        f32x4 aq[4], aw[4], ak[4];  // dQ_S^T, -G_W^T, dK_S^T
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) aq[tt] = aw[tt] = ak[tt] = z4;
        // 32 v at a time: their two waves put their columns of S and dS' into LDS (four
        // planes [v][k], hi and lo), every wave reads its own k of them as rows
        T *const pl = reinterpret_cast<T *>(sR);
        auto hand_on = [&](int kv) {
            if ((w >> 1) != kv) return;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                T *const p = pl + rb[ks & 1] + 16 * (w & 1) * D + 64 * (ks >> 1);
                *reinterpret_cast<frag_t<T> *>(p) = s1h[ks];
                *reinterpret_cast<frag_t<T> *>(p + 32 * D) = s1l[ks];
                *reinterpret_cast<frag_t<T> *>(p + 64 * D) = d1h[ks];
                *reinterpret_cast<frag_t<T> *>(p + 96 * D) = d1l[ks];
            }
            if (nx < items) load_s1(nx);  // (the waves' turns spread these loads over the step)
        };
        if (nx < items) load_regs(xn, gn);
        hand_on(0);
#pragma unroll
        for (int kv = 0; kv < KS; ++kv) {
            __syncthreads();
            auto turned = [&](int plane) { return tr2(pl + plane * 32 * D + tb[0], pl + plane * 32 * D + tb[1]); };
            const frag_t<T> sh = turned(0), sl = turned(1), dh = turned(2), dl = turned(3);
            __syncthreads();  // the planes are read (and, after the last, E1 and E2 may take their place)
            if (kv + 1 < KS) hand_on(kv + 1);
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const frag_t<T> of = rows(sO, tt, kv);
                mma(aq[tt], sh, of);
                mma(aq[tt], sl, of);
                mma3(aw[tt], sh, sl, rows(sGh, tt, kv), rows(sGl, tt, kv));
                mma3(ak[tt], dh, dl, rows(sUh, tt, kv), rows(sUl, tt, kv));
                if (tt & 1) sched_fence();
            }
        }
        positions();

        // --- 3. dA, dP on the causal tiles: rows s = 16 st + 4 q4 + r, column t = 16 tt + n16
        auto tile = [&](int i, bool doA, bool doP) {
            int tt, st;
            tri_tile(i, tt, st);
            f32x4 da = z4, dp = z4, kk = z4, qk = z4;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const frag_t<T> uh = rows(sUh, st, ks), ul = rows(sUl, st, ks), ks4 = rows(sK, st, ks);
                if (doA) {
                    mma3(da, uh, ul, rows(sGh, tt, ks), rows(sGl, tt, ks));
                    mma(kk, ks4, rows(sK, tt, ks));
                }
                if (doP) {
                    const frag_t<T> of = rows(sO, tt, ks);
                    mma(dp, uh, of);
                    mma(dp, ul, of);
                    mma(qk, ks4, rows(sQ, tt, ks));
                }
                sched_fence();
            }
            const int t = 16 * tt + n16, s0 = 16 * st + 4 * q4;
            const float bt = sb[t], be = sbe[t];
            const f32x4 bs = *reinterpret_cast<const f32x4 *>(&sb[s0]);
            f32x4 ah = z4, e1 = z4, exA = z4, exP = z4;
            float rx = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float ga = s0 + r <= t ? fexp2(bt - bs[r]) : 0.f;
                const float dav = s0 + r < t ? -da[r] : 0.f, dpv = s0 + r <= t ? dp[r] : 0.f;
                rx = fmaf(dav, ga * kk[r], rx);  // sum_s dA KK o Gamma (dbeta)
                ah[r] = dav * be * ga;
                e1[r] = dpv * ga;
                exA[r] = ah[r] * kk[r];  // dA o A
                exP[r] = e1[r] * qk[r];  // dP o P
            }
            if (doA) {
                put4(sE2, sE2 + C * C, epos(t, s0), ah);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (s0 + r < t) {
                        const T h = cvt<T>(ah[r]);
                        sE2[epos(s0 + r, t)] = h;
                        sE2[C * C + epos(s0 + r, t)] = cvt<T>(ah[r] - tof<T>(h));
                    }
                rx = sum_rows(rx);
                const float row = sum_rows(exA[0] + exA[1] + exA[2] + exA[3]);
                if (q4 == 0) {
                    sRX[st][t] = rx;
                    sXr[0][st][t] = row;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float c = sum16(exA[r]);
                    if (n16 == 0) sXc[0][tt][s0 + r] = c;
                }
            }
            if (doP) {
                put4(sE1, sE1 + TRI, tri_pos<0>(t, s0), e1);
                const float row = sum_rows(exP[0] + exP[1] + exP[2] + exP[3]);
                if (q4 == 0) sXr[1][st][t] = row;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float c = sum16(exP[r]);
                    if (n16 == 0) sXc[1][tt][s0 + r] = c;
                }
            }
        };
        if constexpr (NW == 8) {  // one tile each; the last two cut in halves over waves 4 to 7
            tile(w, true, true);
            if (w >= 4) tile(8 + ((w >> 1) & 1), w & 1, !(w & 1));
        } else {
            for (int i = w; i < 10; i += NW) tile(i, true, true);
        }
        if (tid < 128) {  // E1's zero blocks (0,1) and (2,3) inside the diagonal quadrants
            const int b = tid >> 6, o = tri_pos<0>(32 * b + ((tid >> 2) & 15), 32 * b + 16 + 4 * (tid & 3));
            *reinterpret_cast<s4v *>(&sE1[o]) = s4v{0, 0, 0, 0};
            *reinterpret_cast<s4v *>(&sE1[TRI + o]) = s4v{0, 0, 0, 0};
        }

        __syncthreads();  // E1, E2 are complete; v's and dO's tiles are free
        if (nx < items) load_vo(xn);

        sched_fence();
        positions();
        // --- 4. dq, dk (rows c = own + r, columns t) and the row sums
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const int t = 16 * tt + n16, p = xb + 16 * tt * D;
            const f32x4 kv = ld4f(sK + p), qv = ld4f(sQ + p);
            float z = 0.f, ww = 0.f, y = 0.f;
            aq[tt] *= sg[t];
            const float et = se[t], bg = sbe[t] * sg[t];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                z = fmaf(-aw[tt][r], kv[r], z);
                ww = fmaf(ak[tt][r], kv[r], ww);
                y = fmaf(qv[r], aq[tt][r], y);
                ak[tt][r] = et * ak[tt][r] - bg * aw[tt][r];
            }
            z = sum_rows(z);
            ww = sum_rows(ww);
            y = sum_rows(y);
            if (q4 == 0) {
                sZ[w][t] = z;
                sW[w][t] = ww;
                sY[w][t] = y;
            }
        }
#pragma unroll
        for (int ks = 0; ks < C / 32; ++ks) {
            const frag_t<T> kf = cols(sK, ks), qf = cols(sQ, ks);
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                if (tt >= 2 * ks) {  // E1[t][s]
                    mma(aq[tt], kf, tri_rows((const short *)sE1, tt, ks));
                    mma(aq[tt], kf, tri_rows((const short *)sE1 + TRI, tt, ks));
                }
                if (tt < 2 * ks + 2) {  // E1[s][t]
                    mma(ak[tt], qf, tri_tr((const short *)sE1, ks, tt));
                    mma(ak[tt], qf, tri_tr((const short *)sE1 + TRI, ks, tt));
                }
                const int o = eb[ks] + 16 * tt * C;
                mma(ak[tt], kf, rd(sE2, o));
                mma(ak[tt], kf, rd(sE2, C * C + o));
            }
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {  // whole rows through U's tiles
            const int p = xb + 16 * tt * D;
            st4(sUh + p, aq[tt][0], aq[tt][1], aq[tt][2], aq[tt][3]);
            st4(sUl + p, ak[tt][0], ak[tt][1], ak[tt][2], ak[tt][3]);
        }
        vm_wait_all();  // this wave's part of the next v and dO is in LDS
        __syncthreads();
        {
            const rsrc_t rq = buf_rsrc((T *)a.dq + xo, span), rk = buf_rsrc((T *)a.dk + xo, span);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int p = sp + i * RS * D;
                buf_st(rq, xoff, i * RS * rowb, *reinterpret_cast<const blk *>(sUh + p));
                buf_st(rk, xoff, i * RS * rowb, *reinterpret_cast<const blk *>(sUl + p));
            }
        }
        if (w == 0) {  // per token t = 63 - lane, so that dg_t = sum_{t' >= t} db_t' is a prefix sum over lanes
            const int t = 63 - lane, tt = t >> 4;
            float gwk = 0.f, dk1 = 0.f, qd = 0.f, guv = 0.f, rx = 0.f, row = 0.f, col = 0.f, tot = 0.f;
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                gwk += sZ[u][t];
                dk1 += sW[u][t];
                qd += sY[u][t];
                guv += sGv[u][t];
                tot += sWav[u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {  // tile columns u <= tt, then tile rows u >= tt (clamped reads, no branches)
                const int lo = u < tt ? u : tt, hi = u > tt ? u : tt;
                const float x = sRX[lo][t], y = sXr[0][lo][t] + sXr[1][lo][t], z = sXc[0][hi][t] + sXc[1][hi][t];
                rx += u <= tt ? x : 0.f;
                row += u <= tt ? y : 0.f;
                col += u >= tt ? z : 0.f;
            }
            a.dbeta[go + (int64_t)t * a.sg_l] = sg[t] * gwk + guv + rx;
            const float rt = se[t] * dk1;
            float db = qd + (row - col) + sbe[t] * sg[t] * gwk - rt;
            const float rsum = lane_value(wave_scan_dpp(rt), 63);
            if (t == C - 1) db += rsum + sg[C - 1] * tot;
            a.dg[go + (int64_t)t * a.sg_l] = wave_scan_dpp(db);
        }
        if (nx >= items) break;
    }
}

template <int D>
hipError_t gdn_phase_d(int phase, const GdnArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const unsigned bh = (unsigned)(a.B * a.H);
    const dim3 wblk(256);
    switch (phase) {
    case GDN_TPREP:
        if constexpr (D == 128)
            hipExtLaunchKernelGGL((k_gdn_tprep<__bf16, D>), dim3((unsigned)(bh * (a.L / C))), wblk, 0, s, e0, e1, 0, a);
        break;
    case GDN_PREP:  // M_J and N_J of 8 items per 16 workgroups
        hipExtLaunchKernelGGL((k_gdn_walk<__bf16, D, W_PREP>), dim3((bh * a.n_prep + 7) / 8 * 16), wblk, 0, s, e0, e1, 0,
                              a);
        break;
    case GDN_SCAN: hipExtLaunchKernelGGL((k_gdn_scan<D>), scan_grid<D>(bh), dim3(4 * D), 0, s, e0, e1, 0, a); break;
    case GDN_OUT:
        if (D == 128 && !a.tw) {
            hipExtLaunchKernelGGL((k_gdn_walk<__bf16, D, W_OUT, false>), dim3(bh * a.n_super), wblk, 0, s, e0, e1, 0, a);
            break;
        }
        hipExtLaunchKernelGGL((k_gdn_walk<__bf16, D, W_OUT>), dim3(bh * a.n_super), wblk, 0, s, e0, e1, 0, a);
        break;
    case GDN_STORE:
        hipExtLaunchKernelGGL((k_gdn_walk<__bf16, D, W_STORE>), dim3(bh * a.n_super), wblk, 0, s, e0, e1, 0, a);
        break;
    case GDN_DPREP:
        hipExtLaunchKernelGGL((k_gdn_dwalk<__bf16, D, true>), dim3(bh * (a.n_super - 1)), wblk, 0, s, e0, e1, 0, a);
        break;
    case GDN_DSCAN: hipExtLaunchKernelGGL((k_gdn_dscan<D>), scan_grid<D>(bh), dim3(4 * D), 0, s, e0, e1, 0, a); break;
    case GDN_DWALK:
        hipExtLaunchKernelGGL((k_gdn_dwalk<__bf16, D, false>), dim3(bh * a.n_super), wblk, 0, s, e0, e1, 0, a);
        break;
    case GDN_DCHUNK: {
        const int64_t items = (int64_t)bh * (a.L / C);
        if (items > 0)
            hipExtLaunchKernelGGL((k_gdn_dchunk<__bf16, D>), dim3((unsigned)std::min<int64_t>(items, a.n_x)),
                                  dim3(4 * D), 0, s, e0, e1, 0, a);
        break;
    }
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

// Argument checks shared by every phase: the superchunk buffers a phase reads
// or writes must be there.
hipError_t launch_gdn_phase(int phase, const GdnArgs &a, int D, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (a.n_super < 1) return hipErrorInvalidValue;
    const bool multi = a.n_super > 1;
    if (D == 128 && phase != GDN_SCAN && phase != GDN_DSCAN && phase != GDN_DCHUNK && a.L >= C && !a.tw &&
        !(phase == GDN_OUT && a.L == C))  // (of one chunk: the walk forms T)
        return hipErrorInvalidValue;
    switch (phase) {
    case GDN_TPREP:
        if (D != 128 || a.L < C) return hipErrorInvalidValue;
        break;
    case GDN_PREP:
    case GDN_SCAN:
        if (!multi || !a.wsS || !a.wsM || !a.wsN || a.n_prep < a.n_super - 1) return hipErrorInvalidValue;
        if (a.scan_out && (a.n_prep != a.n_super || !a.S_out)) return hipErrorInvalidValue;
        break;
    case GDN_DPREP:
    case GDN_DSCAN:
        if (!multi || !a.wsM || !a.wsE || !a.wsDe || a.n_prep != a.n_super) return hipErrorInvalidValue;
        break;
    case GDN_OUT:
        if (multi && !a.wsS) return hipErrorInvalidValue;
        break;
    case GDN_STORE:
        if (!a.wsSc || (multi && !a.wsS)) return hipErrorInvalidValue;
        break;
    case GDN_DWALK:
        if (!a.wsDc || (multi && !a.wsDe)) return hipErrorInvalidValue;
        break;
    case GDN_DCHUNK:
        if (!a.wsSc || !a.wsDc || a.n_x < 1) return hipErrorInvalidValue;
        break;
    default: return hipErrorInvalidValue;
    }
    if (D == 128) return gdn_phase_d<128>(phase, a, s, e0, e1);
    if (D == 64) return gdn_phase_d<64>(phase, a, s, e0, e1);
    return hipErrorInvalidValue;
}

}  // namespace sf
