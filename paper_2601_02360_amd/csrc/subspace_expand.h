// The second product of the subspace calls with its rows held in registers; included by subspace.hip, inside its
// anonymous namespace.
#pragma once

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float vfloat2 __attribute__((ext_vector_type(2)));

// Two floats, each split exactly into three bf16 pieces (packed a low, b high): the first truncated, so that no finite
// float overflows, the second rounded, the third what is left (at most eight significant bits).  Eleven instructions.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
    const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    p0 = pack_bf16(ua, ub);
    const float ra = __fsub_rn(a, __uint_as_float(ua & 0xFFFF0000u)), rb = __fsub_rn(b, __uint_as_float(ub & 0xFFFF0000u));
    p1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(vfloat2{ra, rb}, bf16x2));
    const float sa = __fsub_rn(ra, __uint_as_float(p1 << 16)), sb = __fsub_rn(rb, __uint_as_float(p1 & 0xFFFF0000u));
    p2 = pack_bf16(__float_as_uint(sa), __float_as_uint(sb));
}
__device__ __forceinline__ void split_8(const float (&v)[8], vuint4 (&p)[3]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t q0, q1, q2;
        split_pair(v[2 * i], v[2 * i + 1], q0, q1, q2);
        p[0][i] = q0; p[1][i] = q1; p[2][i] = q2;
    }
}
// acc += A B over 16 k from the pieces of both, smallest terms first
__device__ __forceinline__ v16f mfma_split(const vuint4 (&a)[3], const vuint4 (&b)[3], v16f acc) {
    constexpr int pairs[6][2] = {{2, 0}, {1, 1}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
    for (int c = 0; c < 6; ++c)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[pairs[c][0]]),
                                                      __builtin_bit_cast(bf16x8, b[pairs[c][1]]), acc, 0, 0, 0);
    return acc;
}

// A buffer of `bytes` bytes (below 2^31) from a uniform address: a lane whose offset lies beyond it reads 0 and stores
// nothing, so a lane is left out by adding kNowhere to its offset, without a branch.
typedef __amdgpu_buffer_rsrc_t Buffer;
constexpr uint32_t kNowhere = 0x80000000u;
__device__ __forceinline__ Buffer buffer_of(const float* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, 0x00020000);
}
typedef float valigned4 __attribute__((ext_vector_type(4)));
// The whole offset is the lanes': with a scalar register as offset the compiler lets the instruction behind a 16-byte
// store overwrite the store's data registers, and the store was seen to take the new value (the address of the next one).
template <int AUX>
__device__ __forceinline__ valigned4 buffer_get(Buffer b, uint32_t at) {
    return __builtin_bit_cast(valigned4, __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, AUX));
}
template <int AUX>
__device__ __forceinline__ void buffer_put(Buffer b, uint32_t at, valigned4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(vuint4, v), b, at, 0, AUX);
}
constexpr int kOnce = 2;                         // AUX: non-temporal

// out[M, N] = A U^T (+ epilogue) for row-major A [M, K] and U [N, K], 32 < K <= 32 KS, N > 32: the second
// product of the subspace calls, whose reduction is short and whose output is long.
// LINES: N is a multiple of 32.  Otherwise the last tile begins at column N - 32, so that all of its columns exist -- those it
// shares with the tile before come out the same, from the same operands in the same order, whoever stores them last (code for
// a part of a tile made the compiler spill 70 registers per lane) -- and output and tables go without the non-temporal
// hint: neighbouring tiles share cache lines, which with the hint are fetched twice and written in parts.
//
// gemm_kernel above starts a workgroup per output tile, so that with K = 192 an epilogue that moves up to four arrays
// follows every twelve K tiles, and the operands of a row block are fetched, split and stored to LDS again for every
// column tile.  Here a workgroup of eight waves keeps 128 rows of A in registers -- a wave holds 32 rows and half of K, as
// pieces where products are split -- and walks along the columns, 32 at a time: only U passes through LDS, split once per
// row block, and everything that is not a product sits between the products of the tile that is being multiplied: staging
// of the next U tile, the exchange of the two halves of the previous tile's sums (through LDS, from which it is read back in
// rows, so that a lane finishes four neighbouring columns and whole 128-byte lines are written), its tables requested,
// the tile before that finished.  One barrier a tile, before the last k step, whose operands are in registers by then.
// Two waves per SIMD (256 registers; split products with both tables and k above 192 spill four).
//
// Bound: fp32 by the matrix pipe (79 % busy with both tables at K = 256, 74 % in the update, 2.3 GHz); split products by
// neither pipe alone (51 % busy with both tables at K = 192, 39 % in the update, at 1.8 to 2.0 GHz: splitting, staging and stores sit
// between the products).  Before / now, us: 16384 x 1536 from 192, both tables, split 72.6 / 57.1, fp32 90.9 / 81.7; 16384 x
// 2048 from 256, both tables, fp32 149 / 140; re-projection 41472 x 1792, k 192, split 497 / 442; update at 32000 x 2048 from
// 256, fp32: 320 / 321.  Rows of no whole lines, against the GEMM kernel, one table, split: 3938 x 1291 from 92 36.1 / 25.4,
// 16384 x 1002 from 120 and its like 1.3 times as fast, few rows twice (splc::expand_applies_across_lines).
struct ExpandArgs {
    const float* a;
    const float* u;
    float* out;              // x_hat, or T_S
    float* perp;             // EPI_UPDATE: T_perp
    HighRank h;              // tables of the reconstruction
    int m, n, k;
    int row_blocks, parts;   // of 128 rows; workgroups that share one, or 0 (splc::tile_run)
};
enum { EPI_PERP = 1, EPI_POS = 2, EPI_UPDATE = 4 };

template <int MATH, int KS, int EPI, bool LINES>
__global__ __launch_bounds__(512, 2) void expand_kernel(ExpandArgs g) {
    constexpr int CH = 4 * KS;                   // groups of eight k
    constexpr int NU = (KS + 1) / 2;             // groups of four k of a U tile that a lane stages
    constexpr bool SPLIT = MATH == MATH_BF16X3;
    static_assert(LINES || EPI != EPI_UPDATE, "columns of two tiles would be updated twice");
    constexpr int ONCE = LINES ? kOnce : 0;
    // split: three planes of groups of eight k; fp32: groups of four k, as they are
    __shared__ vuint4 pieces[2][SPLIT ? 3 : 2][CH][33];
    __shared__ valigned4 sums[2][4][2][32][8];   // partial sums of a tile: [row][four columns, their place turned by the row]
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wave & 3, kg = wave >> 2;
    const int M = g.m, N = g.n, K = g.k;

    const int groups = gridDim.x, col_tiles = LINES ? N / 32 : (N + 31) / 32;
    auto column = [&](int t) { return LINES || 32 * t + 32 <= N ? 32 * t : N - 32; };       // first one of a tile
    // neighbouring runs share rows and table lines: each XCD takes a contiguous eighth of them
    const int place = groups % 8 == 0 ? (int)(blockIdx.x & 7) * (groups / 8) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const splc::TileRun run = splc::tile_run(place, groups, g.row_blocks, col_tiles, g.parts);
    int rb = run.row_block, ct = run.col_tile, left = run.tiles;
    if (left == 0) return;

    // Loads of four floats from byte `off` of an array piece that ends at byte `end`: never past the end, and where that
    // moved a load (the last row, K % 4 != 0), `straighten` puts its floats back in place.
    auto straighten = [](vfloat4 v, uint32_t off, uint32_t at) {
        const uint32_t d = (off - at) >> 2;
        vfloat4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w[e] = v[e];
#pragma unroll
            for (int by = 1; by + e < 4; ++by) w[e] = d == (uint32_t)by ? v[e + by] : w[e];
        }
        return w;
    };

    // staging of a U tile: lane t takes the groups of four k number t, t + 512, ... of its 32 rows
    uint32_t u_off[NU];
    vfloat4 raw[NU];
    constexpr auto staged = [](int i, int w) { return (i + 1) * 512 <= 256 * KS || w < 4; };
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int f = tid + 512 * i, n = f / (8 * KS), k0 = 4 * (f % (8 * KS));
        u_off[i] = 4u * (uint32_t)(n * K + (k0 < K ? k0 : 0));
    }
    const bool ragged = (K & 3) != 0;
    auto u_last = [&](int n0) { return (uint32_t)((N - n0 < 33 ? N - n0 : 33) * K - 4) * 4u; };
    auto fetch = [&](int n0) {
        const char* base = reinterpret_cast<const char*>(g.u + (int64_t)n0 * K);
        const uint32_t last = u_last(n0);
#pragma unroll
        for (int i = 0; i < NU; ++i)
            if (staged(i, wave)) raw[i] = *(const SPLC_GLOBAL vfloat4*)(base + (u_off[i] < last ? u_off[i] : last));
    };
    uint32_t half[3];                            // pieces of the first two floats of a group
    auto stash = [&](int i, int part, int n0, int buf) {
        if (!staged(i, wave)) return;
        if (!SPLIT && part == 1) {
            const int f = tid + 512 * i, n = f / (8 * KS), q = f % (8 * KS);
            (&pieces[buf][0][0])[q][n] = __builtin_bit_cast(vuint4, raw[i]);
        } else if (part == 0) {
            if (ragged && n0 + 32 >= N) {
                const uint32_t last = u_last(n0);
                raw[i] = straighten(raw[i], u_off[i], u_off[i] < last ? u_off[i] : last);
            }
            if (K < 32 * KS) {                   // no product with what lies behind a row
                const int k0 = 4 * ((tid + 512 * i) % (8 * KS));
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[i][e] = k0 + e < K ? raw[i][e] : 0.f;
            }
            if (SPLIT) split_pair(raw[i][0], raw[i][1], half[0], half[1], half[2]);
        } else {
            const int f = tid + 512 * i, n = f / (8 * KS), q = f % (8 * KS);
            uint32_t hi[3];
            split_pair(raw[i][2], raw[i][3], hi[0], hi[1], hi[2]);
#pragma unroll
            for (int p = 0; p < 3; ++p)
                reinterpret_cast<vuint2*>(&pieces[buf][p][q >> 1][n])[q & 1] = vuint2{half[p], hi[p]};
        }
    };

    vuint4 a[KS][SPLIT ? 3 : 2];                 // this wave's rows: pieces, or (fp32) k = 16 s + 8 q + 4 h + 0 .. 3 in [s][q]
    uint32_t o_off, t_off[2], p_off[2];          // bytes; a lane finishes four columns of two rows, eight rows apart
    const int fr = 32 * rg + 16 * kg + (lane >> 3), fc = 4 * (lane & 7);
    Buffer out, perp;
    auto take_rows = [&](int b) {
        const int rows = M - b * 128 < 128 ? M - b * 128 : 128, r = 32 * rg + c;
        const char* base = reinterpret_cast<const char*>(g.a + (int64_t)b * 128 * K);
        const uint32_t first_k = (uint32_t)(16 * kg * KS + (SPLIT ? 8 : 4) * h);
        constexpr int STEP = SPLIT ? 4 : 8;      // from a lane's first four k of a step to its other four
        const uint32_t off = 4u * ((uint32_t)(r < rows ? r : rows - 1) * (uint32_t)K + first_k);
        const uint32_t last = 4u * (uint32_t)((M - b * 128 < 129 ? M - b * 128 : 129) * K - 4);
        int width = K;
        asm volatile("" : "+s"(width));          // its comparisons below are made here, not kept in registers over the loop
        int token[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (EPI & EPI_PERP) token[e] = g.h.token[b * 128 + (fr + 8 * e < rows ? fr + 8 * e : rows - 1)];
        vfloat4 v[KS][2];
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t o = off + 64 * s + 4 * STEP * e;
                v[s][e] = *(const SPLC_GLOBAL vfloat4*)(base + (o < last ? o : last));
            }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            float w[8];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t o = off + 64 * s + 4 * STEP * e;
                vfloat4 x = v[s][e];
                if (b * 128 + 128 >= M && (K & 3)) x = straighten(x, o, o < last ? o : last);
#pragma unroll
                for (int i = 0; i < 4; ++i) w[4 * e + i] = (int)first_k + 16 * s + STEP * e + i < width ? x[i] : 0.f;
            }
            if constexpr (SPLIT) {
                split_8(w, a[s]);
            } else {
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    a[s][e] = __builtin_bit_cast(vuint4, vfloat4{w[4 * e], w[4 * e + 1], w[4 * e + 2], w[4 * e + 3]});
            }
        }
        o_off = 4u * (uint32_t)(fr * N + fc);
        out = buffer_of(g.out + (int64_t)b * 128 * N, (uint32_t)(rows * N) * 4u);
        if (EPI == EPI_UPDATE) perp = buffer_of(g.perp + (int64_t)b * 128 * N, (uint32_t)(rows * N) * 4u);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int row = b * 128 + (fr + 8 * e < rows ? fr + 8 * e : rows - 1);
            if (EPI & EPI_PERP) {
                const int t = token[e] < 0 ? 0 : (token[e] >= g.h.vocab ? g.h.vocab - 1 : token[e]);
                t_off[e] = 4u * ((uint32_t)t * (uint32_t)N + (uint32_t)fc);
            }
            if (EPI & EPI_POS) p_off[e] = 4u * ((uint32_t)(row % g.h.seq_len) * (uint32_t)N + (uint32_t)fc);
        }
    };
    valigned4 tab[2][2], part[2][2];
    // rows fr, fr + 8 of a finished tile: the sum of both halves of the reduction, the epilogue, out
    auto put = [&](int e, int n0, bool there) {
        const uint32_t at = o_off + (there ? 32u * (uint32_t)(e * N) + 4u * (uint32_t)n0 : kNowhere);
        valigned4 v, w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = __fadd_rn(part[e][0][i], part[e][1][i]);
            if (EPI == EPI_UPDATE) w[i] = __fadd_rn(tab[1][e][i], __fsub_rn(tab[0][e][i], v[i]));
            if (EPI & EPI_PERP) v[i] = __fadd_rn(v[i], tab[0][e][i]);
            if (EPI & EPI_POS) v[i] = __fadd_rn(v[i], tab[1][e][i]);
        }
        if (EPI == EPI_UPDATE) buffer_put<ONCE>(perp, at, w);
        buffer_put<ONCE>(out, at, v);
    };
    // what put(e) will combine with the product of a tile
    auto request = [&](int e, int n0) {
        if (EPI == EPI_UPDATE) {
            const uint32_t at = o_off + 32u * (uint32_t)(e * N) + 4u * (uint32_t)n0;
            tab[0][e] = buffer_get<ONCE>(out, at);
            tab[1][e] = buffer_get<ONCE>(perp, at);
        } else {
            if (EPI & EPI_PERP) tab[0][e] = *(const SPLC_GLOBAL vfloat4*)((const char*)(g.h.t_perp + n0) + t_off[e]);
            if (EPI & EPI_POS) tab[1][e] = *(const SPLC_GLOBAL vfloat4*)((const char*)(g.h.pos + n0) + p_off[e]);
        }
    };
    // Register v of lane (c, h) is row c, column 8 (v / 4) + 4 h + v % 4 of the tile.
    auto exchange = [&](int slot, const v16f& acc) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            sums[slot][rg][kg][c][(2 * q + h) ^ ((c >> 1) & 7)] = valigned4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    };
    auto receive = [&](int slot) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int r = 16 * kg + 8 * e + (lane >> 3);
#pragma unroll
            for (int p = 0; p < 2; ++p) part[e][p] = sums[slot][rg][p][r][(lane & 7) ^ ((r >> 1) & 7)];
        }
    };

    int buf = 0;
    auto after = [&](int t) { return t + 1 < col_tiles ? t + 1 : 0; };   // past the last tile of all: staged, not used
    fetch(column(ct));
    take_rows(rb);
#pragma unroll
    for (int i = 0; i < NU; ++i) stash(i, 0, column(ct), 0), stash(i, 1, column(ct), 0);
    fetch(column(after(ct)));
    constexpr int NF = SPLIT ? 3 : 2;
    vuint4 f[2][NF];
    auto operands = [&](int b, int s, int set) {
#pragma unroll
        for (int p = 0; p < NF; ++p)
            f[set][p] = SPLIT ? pieces[b][p][2 * (kg * KS + s) + h][c] : (&pieces[b][0][0])[4 * (kg * KS + s) + 2 * p + h][c];
    };
    int from = 0;
    // Tile ct.  Between its products: tile ct + 1 is staged, tile ct + 2 requested; of tile ct - 1 (its sums in `before`)
    // the halves are exchanged and its tables requested; tile ct - 2 is finished.  The barrier comes before the last k
    // step, whose operands are in registers by then; behind it the first operands of the next tile are requested.
    auto tile = [&](v16f& acc, const v16f& before) {
        constexpr int PER = SPLIT ? 6 : 8, NM = PER * KS;      // products per k step, per tile
        const int next = column(after(ct)), second = column(after(after(ct)));
        auto side = [&](int m) {
            // m = 0 .. NM - 1: after product m.
            constexpr int CHUNKS = 3 + 2 * NU;
            const int lo = m * CHUNKS / (NM - PER), hi = (m + 1) * CHUNKS / (NM - PER);
            for (int q = lo; q < hi && q < CHUNKS; ++q) {
                if (q < 2 * NU) {
                    stash(q >> 1, q & 1, next, buf ^ 1);
                    if (q == 2 * NU - 1) fetch(second);
                } else {
                    const int e = q - 2 * NU;
                    if (e < 2) {
                        put(e, 32 * (ct - 2), ct - 2 >= from);
                        request(e, ct - 1 >= from ? 32 * (ct - 1) : 0);
                    } else if (ct - 1 >= from) {
                        exchange((ct - 1) & 1, before);
                    }
                }
            }
        };
        v16f zero;
#pragma unroll
        for (int v = 0; v < 16; ++v) zero[v] = 0.f;
        acc = zero;
        receive(ct & 1);
        constexpr int pairs[6][2] = {{2, 0}, {1, 1}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s + 1 < KS) {
                operands(buf, s + 1, (s + 1) & 1);
            } else {
                __syncthreads();
                operands(buf ^ 1, 0, (s + 1) & 1);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < PER; ++m) {
                if constexpr (SPLIT)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f[s & 1][pairs[m][1]]),
                                                                  __builtin_bit_cast(bf16x8, a[s][pairs[m][0]]), acc, 0, 0, 0);
                else
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(f[s & 1][m >> 2][m & 3]),
                                                               __uint_as_float(a[s][m >> 2][m & 3]), acc, 0, 0, 0);
                if (s + 1 < KS) side(PER * s + m);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (KS & 1) {                            // the next tile's first operands belong into set 0
#pragma unroll
            for (int p = 0; p < NF; ++p) f[0][p] = f[1][p];
        }
        ++ct;
        buf ^= 1;
    };
    __syncthreads();
    operands(0, 0, 0);
    for (;;) {
        const int until = col_tiles - ct < left ? col_tiles : ct + left;
        left -= until - ct;
        from = ct;
        v16f acc0, acc1;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc0[v] = acc1[v] = 0.f;
        for (;;) {
            tile(acc0, acc1);
            if (ct == until) {
                acc1 = acc0;
                break;
            }
            tile(acc1, acc0);
            if (ct == until) break;
        }
        // the last two tiles
        receive(ct & 1);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            put(e, 32 * (ct - 2), ct - 2 >= from);
            request(e, column(ct - 1));
        }
        exchange((ct - 1) & 1, acc1);
        __syncthreads();
        receive((ct - 1) & 1);
#pragma unroll
        for (int e = 0; e < 2; ++e) put(e, column(ct - 1), true);
        if (left == 0) return;
        take_rows(++rb);
        ct = 0;
    }
}

template <int MATH, int EPI, bool LINES>
void launch_expand(const ExpandArgs& g, int groups, hipStream_t st) {
    const dim3 grid((unsigned)groups), block(512);
    auto run = [&](auto steps) {
        constexpr int KS = decltype(steps)::value;
        constexpr int tables = (EPI & EPI_PERP ? 1 : 0) + (EPI & EPI_POS ? 1 : 0);
        constexpr bool split = MATH == MATH_BF16X3;
        if constexpr (LINES ? splc::expand_takes_steps(KS, tables, EPI == EPI_UPDATE, split)
                            : splc::expand_takes_steps_across_lines(KS, tables, split))
            hipLaunchKernelGGL((expand_kernel<MATH, KS, EPI, LINES>), grid, block, 0, st, g);
    };
    switch ((g.k + 31) / 32) {
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        case 7: run(std::integral_constant<int, 7>{}); break;
        case 8: run(std::integral_constant<int, 8>{}); break;
    }
}
// units: compute units, each of which holds one workgroup
template <int EPI>
void launch_expand(ExpandArgs g, int matmul, int units, hipStream_t st) {
    const int col_tiles = (g.n + 31) / 32;
    g.row_blocks = (g.m + 127) / 128;
    g.parts = splc::parts_of_row_block(g.row_blocks, col_tiles, units);
    const int64_t tiles = (int64_t)g.row_blocks * col_tiles;
    const int groups = g.parts ? g.parts * g.row_blocks : (int)(tiles < units ? tiles : units);
    const bool split = matmul == SPLC_MATMUL_BF16X3;
    if constexpr (EPI != EPI_UPDATE) {           // (splc::expand_applies asks for whole lines there)
        if (g.n % 32 != 0) {
            if (split) launch_expand<MATH_BF16X3, EPI, false>(g, groups, st);
            else launch_expand<MATH_F32, EPI, false>(g, groups, st);
            return;
        }
    }
    if (split) launch_expand<MATH_BF16X3, EPI, true>(g, groups, st);
    else launch_expand<MATH_F32, EPI, true>(g, groups, st);
}
