// The first product of the subspace calls for blocks of 64 rows, split products and fp32; included by subspace.hip, inside its
// anonymous namespace, after subspace_expand.h.
#pragma once

// out[rows, k] = (x - T_perp[token] - PosEmbed) U with 64 < k <= 192, every product split.
//
// gemm_kernel covers 192 columns with three workgroups per 64 rows, each of which gathers, subtracts and splits the same
// rows, and splits, stores, waits and multiplies one after the other.  Here a workgroup of eight waves takes all columns of 64
// rows.  Four pairs of waves share the reduction, a k step of 16 each of a round of 64; a wave of a pair has all 64 rows and
// half of the columns, so a piece that it reads from LDS feeds two or three products.  A goes through LDS, split once by the
// pair; U needs none, since only one wave uses what it loads: its eight k of NJ neighbouring columns come from global
// memory in the layout of the MFMA (the permutation of columns that this makes is undone by the sum at the end) and are
// split tile by tile.  Splitting, staging and the requests of the next rounds sit between the products; one barrier a round.
// The four partial sums are added through LDS in the order of k steps.  Two waves per SIMD (256 registers: requesting A two
// rounds ahead instead of one does not fit and gains nothing where it does; with both tables at NJ = 3 two registers are spilled).
//
// Bound: neither pipe alone: matrix pipes 49 ... 56 % busy at 1.75 to 1.85 GHz (fp32 products: 2.3 GHz), the vector ALU splits
// beside them.  GEMM kernel / this, us: 16384 x 1536 onto 192, no tables 78 / 58, both 93 / 65;
// onto 128: 61 / 40, 60 / 49; 31813 x 1791 onto 182, both tables: 335 / 183; 44032 x 1324 onto 175: 188 / 141.

struct ContractArgs {
    const float* x;
    const float* u;          // [d, k]
    float* out;              // [rows, k]
    HighRank h;
    int rows, d, k;
};

// The four partial sums of each element meet in LDS, 32 rows at a time, and are added in the order of the shares.
template <int NJ>
__device__ __forceinline__ void add_shares(float (&sums)[8][32][32 * NJ], const v16f (&acc)[2][NJ], const ContractArgs& g,
                                           int m0, int rows, int wave, int h, int col, int tid) {
    constexpr int KG = 4, WIDE = 32 * NJ;
    const int first = WIDE * (wave & 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float* const at = &sums[wave][8 * (v >> 2) + 4 * h + (v & 3)][0];
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (col + j >= first) at[col + j - first] = acc[i][j][v];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 32 * 2 * WIDE / 512; ++e) {
            const int f = tid + 512 * e, row = f / (2 * WIDE), cc = f % (2 * WIDE), side = cc / WIDE;
            float sum = sums[side][row][cc - WIDE * side];
#pragma unroll
            for (int p = 1; p < KG; ++p) sum = __fadd_rn(sum, sums[2 * p + side][row][cc - WIDE * side]);
            if (32 * i + row < rows && cc < g.k) g.out[(int64_t)(m0 + 32 * i + row) * g.k + cc] = sum;
        }
    }
}

template <int NJ, bool TP, bool PE>
__global__ __launch_bounds__(512, 2) void contract_kernel(ContractArgs g) {
    constexpr int KG = 4, DEEP = 16 * KG;        // k steps of 16 that a round covers, one per pair of waves
    constexpr int WIDE = 32 * NJ;                // columns of a wave
    typedef float vcols __attribute__((ext_vector_type(NJ), aligned(4)));
    union Shared {
        vuint4 a[2][KG][3][2][65];               // pieces: [half of a step][row]
        float sums[8][32][WIDE];
    };
    __shared__ __attribute__((aligned(16))) Shared sm;
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = wave & 1, kg = wave >> 1;
    const int d = g.d, N = g.k;
    const int m0 = blockIdx.x * 64, rows = g.rows - m0 < 64 ? g.rows - m0 : 64;

    // A: the two waves of a step take 32 rows each, a lane eight k of one
    const int ar = 32 * cg + (lane >> 1), ah = lane & 1;
    const int arow = m0 + (ar < rows ? ar : rows - 1);
    const char* const xb = reinterpret_cast<const char*>(g.x + (int64_t)m0 * d);
    const uint32_t x_off = 4u * ((uint32_t)(arow - m0) * (uint32_t)d + 8u * (uint32_t)ah);
    uint32_t t_off = 0, p_off = 0;
    if (TP) {
        int t = g.h.token[arow];
        t = t < 0 ? 0 : (t >= g.h.vocab ? g.h.vocab - 1 : t);
        t_off = 4u * ((uint32_t)t * (uint32_t)d + 8u * (uint32_t)ah);
    }
    if (PE) p_off = 4u * ((uint32_t)(arow % g.h.seq_len) * (uint32_t)d + 8u * (uint32_t)ah);
    // B: a lane holds columns col .. col + NJ - 1 of its wave's, at eight k.  A lane beyond column N, or across it, takes the
    // last NJ columns, which another lane has too.
    const int col = WIDE * cg + NJ * c < N - NJ ? WIDE * cg + NJ * c : N - NJ;
    const uint32_t u_off = 4u * (uint32_t)(8 * h * N + col), u_last = 4u * ((uint32_t)(d - 1) * (uint32_t)N + (uint32_t)col);

    struct StageA { vfloat4 x[2], t[2], p[2]; };
    StageA sa;
    vcols b0[8], b1[8];
    const int rounds = (d + DEEP - 1) / DEEP, plain_rounds = d / DEEP;
    auto fetch_a = [&](auto plain, int r) {
        const int k0 = (r * KG + kg) * 16;
        if (decltype(plain)::value || k0 + 16 <= d) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t at = 4u * (uint32_t)k0 + 16u * e;
                sa.x[e] = *(const SPLC_GLOBAL vfloat4*)(xb + at + x_off);
                if (TP) sa.t[e] = *(const SPLC_GLOBAL vfloat4*)((const char*)g.h.t_perp + at + t_off);
                if (PE) sa.p[e] = *(const SPLC_GLOBAL vfloat4*)((const char*)g.h.pos + at + p_off);
            }
        } else {                                 // zeros from k = d on
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                sa.x[e] = vfloat4{0.f, 0.f, 0.f, 0.f};
                if (TP) sa.t[e] = sa.x[e];
                if (PE) sa.p[e] = sa.x[e];
            }
            if (k0 >= d) return;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool there = k0 + 8 * ah + i < d;
                const uint32_t at = there ? 4u * (uint32_t)(k0 + i) : 0u - 32u * (uint32_t)ah;
                const float vx = *(const SPLC_GLOBAL float*)(xb + (x_off + at));
                sa.x[i >> 2][i & 3] = there ? vx : 0.f;
                if (TP) {
                    const float vt = *(const SPLC_GLOBAL float*)((const char*)g.h.t_perp + (t_off + at));
                    sa.t[i >> 2][i & 3] = there ? vt : 0.f;
                }
                if (PE) {
                    const float vp = *(const SPLC_GLOBAL float*)((const char*)g.h.pos + (p_off + at));
                    sa.p[i >> 2][i & 3] = there ? vp : 0.f;
                }
            }
        }
    };
    auto fetch_b = [&](auto plain, int r, int t, vcols& q) {      // row 8 h + t of this wave's step
        const int k0 = (r * KG + kg) * 16;
        if (decltype(plain)::value) {
            q = *(const SPLC_GLOBAL vcols*)((const char*)(g.u + (int64_t)(k0 + t) * N) + u_off);
        } else {                                 // from row d on the last row: A is zero there
            const uint32_t at = u_off + 4u * (uint32_t)(k0 + t) * (uint32_t)N;
            q = *(const SPLC_GLOBAL vcols*)((const char*)g.u + (at < u_last ? at : u_last));
        }
    };
    // pair `i` of this lane's eight k: tables applied, split, to LDS with the last
    vuint2 put[3];
    auto stash = [&](int i, int buf) {
        float v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int n = 2 * i + e;
            v[e] = sa.x[n >> 2][n & 3];
            if (TP) v[e] = __fsub_rn(v[e], sa.t[n >> 2][n & 3]);
            if (PE) v[e] = __fsub_rn(v[e], sa.p[n >> 2][n & 3]);
        }
        uint32_t p0, p1, p2;
        split_pair(v[0], v[1], p0, p1, p2);
        put[0][i & 1] = p0; put[1][i & 1] = p1; put[2][i & 1] = p2;
        if (i & 1) {
#pragma unroll
            for (int p = 0; p < 3; ++p) reinterpret_cast<vuint2*>(&sm.a[buf][kg][p][ah][ar])[i >> 1] = put[p];
        }
    };

    v16f acc[2][NJ];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    vuint4 fa[2][3];
    auto rows_of = [&](int buf, int i, int p) { fa[i][p] = sm.a[buf][kg][p][h][32 * i + c]; };
    vuint4 pb[2][3];                             // pieces of a column tile, two tiles deep
    auto split_b = [&](int i, int j, const vcols (&b)[8], int set) {     // pair i of column tile j
        uint32_t p0, p1, p2;
        split_pair(b[2 * i][j], b[2 * i + 1][j], p0, p1, p2);
        pb[set][0][i] = p0; pb[set][1][i] = p1; pb[set][2][i] = p2;
    };

    // One round.  Between its products: A of round r + 1 goes to LDS, A and B of round r + 2 are requested, and the next
    // column tile of U is split.  The barrier comes before the last column tile; behind it the rows of the next round are
    // read as those of this one are done with.
    auto one_round = [&](auto plain, int r, auto parity, vcols (&now)[8], vcols (&next)[8]) {
        constexpr int buf = decltype(parity)::value;
        constexpr int pairs[6][2] = {{2, 0}, {1, 1}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};
        constexpr int ODD = NJ & 1;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int set = (j + (ODD ? buf : 0)) & 1;
            if (j == NJ - 1) __syncthreads();
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int m = 0; m < 6; ++m) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[i][pairs[m][0]]),
                                                                        __builtin_bit_cast(bf16x8, pb[set][pairs[m][1]]),
                                                                        acc[i][j], 0, 0, 0);
                    const int n = 6 * i + m;
                    if (n % 3 == 1) {
                        if (j + 1 < NJ) split_b(n / 3, j + 1, now, set ^ 1);
                        else split_b(n / 3, 0, next, set ^ 1);
                    }
                    if (j < NJ - 1) {            // A of the next round, over the tiles before the barrier
                        constexpr int SLOTS = 12 * (NJ - 1);
                        const int at = 12 * j + n;
                        if (at % (SLOTS / 4) == SLOTS / 4 - 1) stash(at / (SLOTS / 4), buf ^ 1);
                        if (at == SLOTS - 1 && (decltype(plain)::value || r + 2 < rounds)) fetch_a(plain, r + 2);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (j == NJ - 1) {
#pragma unroll
                    for (int p = 0; p < 3; ++p) rows_of(buf ^ 1, i, p);
                    if (i == 0 && (decltype(plain)::value || r + 2 < rounds)) {
#pragma unroll
                        for (int t = 0; t < 8; ++t) fetch_b(plain, r + 2, t, now[t]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };
    const std::integral_constant<bool, true> plain;
    const std::integral_constant<bool, false> any;
    fetch_a(any, 0);
#pragma unroll
    for (int t = 0; t < 8; ++t) fetch_b(any, 0, t, b0[t]);
#pragma unroll
    for (int i = 0; i < 4; ++i) stash(i, 0);
    fetch_a(any, 1);                             // (zeros, and the last row of U, if there is no second round)
#pragma unroll
    for (int t = 0; t < 8; ++t) fetch_b(any, 1, t, b1[t]);
#pragma unroll
    for (int i = 0; i < 4; ++i) split_b(i, 0, b0, 0);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p) rows_of(0, i, p);
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    int r = 0;
    for (; r + 3 < plain_rounds; r += 2) {
        one_round(plain, r, even, b0, b1);
        one_round(plain, r + 1, odd, b1, b0);
    }
    for (; r < rounds; r += 2) {
        one_round(any, r, even, b0, b1);
        if (r + 1 < rounds) one_round(any, r + 1, odd, b1, b0);
    }
    add_shares<NJ>(sm.sums, acc, g, m0, rows, wave, h, col, tid);
}

// The same with fp32 products, 128 < k <= 256: the row blocks, column halves and shares of the reduction are those of
// contract_kernel, a round is 64 k, a share two groups of 8.  Lane half h takes k 4 h .. 4 h + 3 of a group, and product t
// multiplies the set {t, 4 + t}, so that a lane reads its row of A as 16 bytes and needs four rows of U.  A row of U is
// requested anew as soon as its products are issued, x and its tables a round ahead, 256 bytes of a row at a time.
//
// Bound: the fp32 matrix pipe (at 16384 x 2048 onto 256 no tables 133 us of at least 109; with both tables 78 % busy at
// 2.3 GHz).  The GEMM kernel gathers and
// subtracts a row twice and pads 129 ... 192 columns to 256.  GEMM kernel / this, us, one card: 16384 x 2048 onto 256, both tables
// 168 / 146; 16384 x 1536 onto 192: 97 / 85; 32768 x 2048 onto 256: 309 / 293; without tables 132 / 133.  128 bytes of a row
// at a time: 156; the order of all instructions fixed: 169; free over a whole group instead of half a group: 151 to 146.
template <int NJ, bool TP, bool PE>
__global__ __launch_bounds__(512, 2) void contract_fp32_kernel(ContractArgs g) {
    constexpr int KG = 4, DEEP = 16 * KG;        // a round: 16 k for every pair of waves
    constexpr int WIDE = 32 * NJ;                // columns of a wave
    typedef float v4f __attribute__((ext_vector_type(4)));
    typedef float vcols __attribute__((ext_vector_type(NJ), aligned(4)));
    union Shared {
        v4f a[2][4 * KG][65];                    // [four k][row]; the pitch spreads writes and reads over all banks
        float sums[8][32][WIDE];
    };
    __shared__ __attribute__((aligned(16))) Shared sm;
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = wave & 1, kg = wave >> 1;
    const int d = g.d, N = g.k;
    const int m0 = blockIdx.x * 64, rows = g.rows - m0 < 64 ? g.rows - m0 : 64;

    // A: sixteen threads take 256 bytes of a row, four k each, of two rows
    const int ar = tid >> 4, aq = tid & 15;
    const char* const xb = reinterpret_cast<const char*>(g.x + (int64_t)m0 * d);
    uint32_t x_off[2], t_off[2], p_off[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int row = ar + 32 * e < rows ? ar + 32 * e : rows - 1;
        x_off[e] = 4u * ((uint32_t)row * (uint32_t)d + 4u * (uint32_t)aq);
        if (TP) {
            int t = g.h.token[m0 + row];
            t = t < 0 ? 0 : (t >= g.h.vocab ? g.h.vocab - 1 : t);
            t_off[e] = 4u * ((uint32_t)t * (uint32_t)d + 4u * (uint32_t)aq);
        }
        if (PE) p_off[e] = 4u * ((uint32_t)((m0 + row) % g.h.seq_len) * (uint32_t)d + 4u * (uint32_t)aq);
    }
    // B: columns as in contract_kernel
    const int col = WIDE * cg + NJ * c < N - NJ ? WIDE * cg + NJ * c : N - NJ;
    const uint32_t u_off = 4u * (uint32_t)(4 * h * N + col);

    struct StageA { vfloat4 x, t, p; };
    StageA sa[2];
    vcols b[2][4];
    const int rounds = (d + DEEP - 1) / DEEP, plain_rounds = d / DEEP;
    auto fetch_a = [&](auto plain, int r) {
        const int k0 = r * DEEP;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            StageA& s = sa[e];
            if (decltype(plain)::value || k0 + DEEP <= d) {
                const uint32_t at = 4u * (uint32_t)k0;
                s.x = *(const SPLC_GLOBAL vfloat4*)(xb + at + x_off[e]);
                if (TP) s.t = *(const SPLC_GLOBAL vfloat4*)((const char*)g.h.t_perp + at + t_off[e]);
                if (PE) s.p = *(const SPLC_GLOBAL vfloat4*)((const char*)g.h.pos + at + p_off[e]);
            } else {                             // zeros from k = d on
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool there = k0 + 4 * aq + i < d;
                    const uint32_t at = there ? 4u * (uint32_t)(k0 + i) : 0u - 16u * (uint32_t)aq;
                    const float vx = *(const SPLC_GLOBAL float*)(xb + (x_off[e] + at));
                    s.x[i] = there ? vx : 0.f;
                    if (TP) {
                        const float vt = *(const SPLC_GLOBAL float*)((const char*)g.h.t_perp + (t_off[e] + at));
                        s.t[i] = there ? vt : 0.f;
                    }
                    if (PE) {
                        const float vp = *(const SPLC_GLOBAL float*)((const char*)g.h.pos + (p_off[e] + at));
                        s.p[i] = there ? vp : 0.f;
                    }
                }
            }
        }
    };
    auto fetch_b = [&](auto plain, int r, int q, int t) {         // row 4 h + t of group q of this wave's share
        const int k0 = r * DEEP + 16 * kg + 8 * q + t;
        if (decltype(plain)::value) {
            b[q][t] = *(const SPLC_GLOBAL vcols*)((const char*)(g.u + (int64_t)k0 * N) + u_off);
        } else {                                 // zeros from row d on
            const bool there = k0 + 4 * h < d;
            b[q][t] = *(const SPLC_GLOBAL vcols*)(g.u + ((int64_t)(there ? k0 + 4 * h : d - 1) * N + col));
#pragma unroll
            for (int j = 0; j < NJ; ++j) b[q][t][j] = there ? b[q][t][j] : 0.f;
        }
    };
    auto stash = [&](int e, int buf) {
        v4f v;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = sa[e].x[i];
            if (TP) v[i] = __fsub_rn(v[i], sa[e].t[i]);
            if (PE) v[i] = __fsub_rn(v[i], sa[e].p[i]);
        }
        sm.a[buf][aq][ar + 32 * e] = v;
    };

    v16f acc[2][NJ];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    v4f fa[2][2];                                // [group][half of the rows]
    auto rows_of = [&](int buf, int q) {
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[q][i] = sm.a[buf][4 * kg + 2 * q + h][32 * i + c];
    };

    // One round.  With its first group A of round r + 1 goes to LDS and that of round r + 2 is requested; the barrier comes
    // between the groups, and behind it the first group of round r + 1 is read.
    auto one_round = [&](auto plain, int r, auto parity) {
        constexpr int buf = decltype(parity)::value;
        rows_of(buf, 1);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (q == 1) {
                __syncthreads();
                rows_of(buf ^ 1, 0);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[q][i][t], b[q][t][j], acc[i][j], 0, 0, 0);
                        if (q == 0 && t == 0 && j == 0) stash(i, buf ^ 1);
                        if (q == 0 && t == 0 && j == 1 && i == 0 && (decltype(plain)::value || r + 2 < rounds))
                            fetch_a(plain, r + 2);
                    }
                if (decltype(plain)::value || r + 1 < rounds) fetch_b(plain, r + 1, q, t);
                if (t & 1) __builtin_amdgcn_sched_barrier(0);    // the compiler orders half a group
            }
        }
    };
    const std::integral_constant<bool, true> plain;
    const std::integral_constant<bool, false> any;
    fetch_a(any, 0);
#pragma unroll
    for (int t = 0; t < 8; ++t) fetch_b(any, 0, t >> 2, t & 3);
    stash(0, 0);
    stash(1, 0);
    fetch_a(any, 1);                             // (zeros if there is no second round)
    __syncthreads();
    rows_of(0, 0);
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    int r = 0;
    for (; r + 3 < plain_rounds; r += 2) {
        one_round(plain, r, even);
        one_round(plain, r + 1, odd);
    }
    for (; r < rounds; r += 2) {
        one_round(any, r, even);
        if (r + 1 < rounds) one_round(any, r + 1, odd);
    }
    add_shares<NJ>(sm.sums, acc, g, m0, rows, wave, h, col, tid);
}

template <int NJ, bool SPLIT>
void launch_contract(const ContractArgs& g, hipStream_t st) {
    const dim3 grid((unsigned)((g.rows + 63) / 64)), block(512);
    auto run = [&](auto tp, auto pe) {
        constexpr bool TP = decltype(tp)::value, PE = decltype(pe)::value;
        if constexpr (!splc::contract_takes_columns(NJ, TP + PE, SPLIT)) return;
        else if constexpr (SPLIT) hipLaunchKernelGGL((contract_kernel<NJ, TP, PE>), grid, block, 0, st, g);
        else hipLaunchKernelGGL((contract_fp32_kernel<NJ, TP, PE>), grid, block, 0, st, g);
    };
    const std::true_type yes;
    const std::false_type no;
    if (g.h.t_perp && g.h.pos) run(yes, yes);
    else if (g.h.t_perp) run(yes, no);
    else if (g.h.pos) run(no, yes);
    else run(no, no);
}
void launch_contract(const ContractArgs& g, bool split, hipStream_t st) {
    if (split) {
        if (g.k <= 128) launch_contract<2, true>(g, st);
        else launch_contract<3, true>(g, st);
    } else if (g.k <= 192) launch_contract<3, false>(g, st);
    else launch_contract<4, false>(g, st);
}
