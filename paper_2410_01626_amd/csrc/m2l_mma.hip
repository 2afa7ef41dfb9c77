// m2l_mma.hip -- FP32 and FP64 M2L on the matrix cores.
//
// lambda~_t = sum over the 189 offsets of T(o) mu~_{t - o}, as products of one
// K x K operator with 16 source expansions at a time
// (v_mfma_f32_16x16x4_f32 / v_mfma_f64_16x16x4_f64: A lane l holds
// A[l % 16][l / 16], B lane l holds B[l / 16][l % 16]; FP32 output lane l holds
// D[4 (l / 16) + v][l % 16], FP64 D[4 v + l / 16][l % 16]).
//
// What bounds it: the matrix cores (FP64: 30 tiles of 21 products of 64 cycles
// per offset and 80 columns at p = 8); the operators (65 KB each in FP64) and
// the source rows have to arrive behind them.  So
//  - operators are stored as their own LDS images and copied straight to LDS
//    (global_load_lds), two buffers, one wait and one barrier per offset;
//  - source rows never touch LDS: a lane needs 16-byte pieces of one row
//    (B fragments of different columns share nothing), which go to registers,
//    the next offset's while this one is multiplied;
//  - a wavefront takes 16 columns and all row tiles of its work-group, so that
//    a source row is fetched and signed once (with two row tiles per wavefront
//    the L1 lookups of the scattered rows took as long as the products).
// All classes use class 0's 189 operators through the reflections of the axes
// (T(P o) = S T(o) S, exactly): S flips the sign bits of the source fragments
// and of the result rows.  FP64 work-groups mix the columns of all classes and
// replicas (a small tree fills its 16-column groups that way, and an operator
// is read once for all of them); FP32 work-groups take one class and run
// through the offsets in that class's own order, chunk by chunk, so that every
// sum is formed in the order of the class's offset list.
//
// Measured (launch; before: operators and sources staged through registers into
// LDS, two barriers per offset): 30,000-atom box at depth 3, p = 8: FP64 166 ->
// 51 us (28.6 TFLOP/s; the products alone take 36 us, 40% of them padding of
// rows, columns and chunks), FP32 94 -> 43 us; 1,000 open atoms at depth 2,
// p = 6, FP32 43 -> 15 us (eleven offsets in a row at a memory latency each);
// 2,300 atoms at depth 2, p = 10, FP64 (a block per target box before) 1,804 ->
// 26 us.  Tried: two row tiles per wavefront throughout (FP64 53, FP32 48-54 us),
// copies and loads spread between the products (FP64 54, FP32 47 us).

namespace fmmk {

// Compile-time sizes of the matrix-core M2L at order P in type T.
template <typename T, int P>
struct MmaDims {
    static constexpr int K = (P + 1) * (P + 1);
    static constexpr int KP = (K + 3) & ~3;        // contraction length
    static constexpr int NF = KP / 16;             // whole chunks of 16 k
    static constexpr int NT = (KP % 16) / 4;       // k-steps of 4 in the tail
    static constexpr int RT = (K + 15) / 16;       // row tiles
    // Row tiles of one work-group.  FP32: half of them (all up to three), so
    // that the work-groups are short and share CUs (a class's offsets fall
    // unevenly into the chunks: 0 to 11 of them).  FP64: as many as two operator
    // buffers in at most 144 KB of LDS hold.
    static constexpr int kTileBytes = 16 * KP * (int)sizeof(T);
    static constexpr int kLds = 73728 / kTileBytes;
    static constexpr int kHalf = RT <= 3 ? RT : (RT + 1) / 2;
    static constexpr int kFit = sizeof(T) == 4 && kHalf < kLds ? kHalf : kLds;
    static constexpr int NPART = (RT + kFit - 1) / kFit;
    static constexpr int RTB = (RT + NPART - 1) / NPART;
    static constexpr int kGroups = sizeof(T) == 4 ? 5 : 4;  // 16-column groups per work-group, at most
    // Row tiles of one wavefront: all of the work-group's (a source row is then
    // fetched and signed once for all of them), or for small FP64 trees two
    // (four SIMDs share the rows of a few columns)
    static constexpr int kNarrow = sizeof(T) == 8 && RTB > 2 && RTB % 2 == 0 ? 2 : RTB;
    // Column groups of a work-group that sums the chunks itself (kSeq): as many
    // as the registers allow
    static constexpr int kSeqGroups = RTB / kNarrow > 2 || (RTB / kNarrow == 2 && KP > 112) ? 2 : kGroups;
    static constexpr int RPB = 16 * RTB;           // operator rows of a part
    // 16-byte chunks of a part's image, in whole wavefront copies
    static constexpr int a_chunks = (RPB * KP * (int)sizeof(T) / 16 + 63) & ~63;
    static_assert(16 * NF <= K, "a whole chunk holds only stored coefficients");
    static_assert(kFit >= 1 && 2 * a_chunks * 16 + (2 * K + kTreeThreads) * 8 <= (int)kLdsBytes, "two operator buffers fit the LDS");
};

// Element of operator entry (row, k) in a part's LDS image; row counts from
// the part's first row.  Whole chunks hold 16-byte pieces per (kc, kq, row):
// FP32 lane group kq takes k = 16 kc + 4 s + kq for s = 0..3 (the products then
// run over k in order), FP64 k = 16 kc + 8 h + 2 kq + e for s = 2 h + e (the
// 16-byte pieces of the four lane groups are then one run of 64 bytes of the
// source row).  The tail holds one element per (s, kq, row), k = 16 NF + 4 s + kq.  FP64 rows are
// stored at the position whose output register order is the row order.
template <typename T>
inline size_t mma_image_index(int RPB, int NF, int row, int k) {
    const int r16 = row & 15;
    const int rr = sizeof(T) == 8 ? (row & ~15) + 4 * (r16 & 3) + (r16 >> 2) : row;
    if (k < 16 * NF) {
        const int kc = k >> 4;
        if (sizeof(T) == 4) return ((size_t)(kc * 4 + (k & 3)) * RPB + rr) * 4 + ((k >> 2) & 3);
        return (((size_t)(kc * 4 + ((k >> 1) & 3)) * 2 + ((k >> 3) & 1)) * RPB + rr) * 2 + (k & 1);
    }
    return (size_t)16 * NF * RPB + (size_t)(k - 16 * NF) * RPB + rr;
}

struct MmaArgs {
    int32_t R;        // replicas
    int32_t ncol;     // target columns per class (all levels)
    int32_t merged;   // 1: columns of all classes and replicas in one list
    int32_t nchunk;   // offset chunks (kSeq: chunks to sum in registers)
    int64_t nt_all;   // boxes at levels >= lmin (partial-buffer stride)
};

template <typename T> struct MmaAcc;
template <> struct MmaAcc<float> { using type = mf4; };
template <> struct MmaAcc<double> { using type = md4; };
__device__ __forceinline__ mf4 mma4(float a, float b, mf4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ md4 mma4(double a, double b, md4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// v with its sign flipped when bit `bit` of m is set
__device__ __forceinline__ float flip(float v, uint64_t m, int bit) {
    const uint32_t h = (uint32_t)(m >> (bit & 32));
    return __uint_as_float(__float_as_uint(v) ^ ((h << (31 - (bit & 31))) & 0x80000000u));
}
__device__ __forceinline__ double flip(double v, uint64_t m, int bit) {
    const uint32_t h = (uint32_t)(m >> (bit & 32));
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, u ^ ((uint64_t)((h << (31 - (bit & 31))) & 0x80000000u) << 32));
}

// Transpose of four registers over the four 16-lane rows of a wavefront:
// register s of row q receives register q of row s.
__device__ __forceinline__ void transpose_rows(float (&r)[4]) {
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = __float_as_uint(r[i]);
    auto a = __builtin_amdgcn_permlane32_swap(u[0], u[2], false, false);
    auto b = __builtin_amdgcn_permlane32_swap(u[1], u[3], false, false);
    auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    r[0] = __uint_as_float(c[0]);
    r[1] = __uint_as_float(c[1]);
    r[2] = __uint_as_float(d[0]);
    r[3] = __uint_as_float(d[1]);
}

// One work-group: one task (row part, chunk of offsets; FP32: one class) and
// one tile of up to kGroups 16-column groups (grid y, and z past the 65,536
// blocks that y may have: 15 FP64 systems at depth 6 make 70,217 tiles).  Wavefront w
// takes column group w / NRG and row tiles RTW (w % NRG) ...
// olist entries: operator slot << 16 | canonical offset index.  masks[cls][kq]:
// the reflection signs of class cls as bits: [0] bit i for the lane's i-th
// source coefficient of the whole chunks, [1] bit s for tail coefficient
// 16 NF + 4 s + kq, [2] bit 4 rt + v for row 16 rt + 4 kq + v.
//
// kSeq: one work item runs through every offset and adds the nchunk chunks' sums
// itself, in m2l_chunk_sum's order (four interleaved sums in registers), so that
// a workspace without room for partials gives the same bits (FP64, p = 9, depth
// 3, chunks of one offset: 700 us an evaluation against 240 with partials).
template <typename T, int P, int RTW, bool kSeq = false>
__global__ __launch_bounds__((64 * (kSeq ? MmaDims<T, P>::kSeqGroups : MmaDims<T, P>::kGroups) * (MmaDims<T, P>::RTB / RTW))) void k_m2l_mma(
    Geo g, MmaArgs ma, const M2LTask* __restrict__ tasks, const int32_t* __restrict__ olist,
    const T* __restrict__ mult_all, const T* __restrict__ zrow, const uint4* __restrict__ bank,
    const uint64_t* __restrict__ masks, T* __restrict__ loc_all, T* __restrict__ part_all, RootArgs ra) {
    using D = MmaDims<T, P>;
    constexpr int NF = D::NF, NT = D::NT, RPB = D::RPB, NRG = D::RTB / RTW;
    constexpr int E = 16 / (int)sizeof(T);  // elements of a 16-byte piece
    // two distinct objects: the copy into one provably leaves the other alone
    __shared__ uint4 op0[D::a_chunks], op1[D::a_chunks];
    const int tile = (int)(blockIdx.z * gridDim.y + blockIdx.y);
    if (ra.root_l && blockIdx.x + 1 == gridDim.x) {
        // the extra last work-groups of a periodic tree form the root's local
        // expansion from the level-1 shares (each of them some replicas')
        __shared__ double rt[2 * D::K + kTreeThreads];
        for (int r = tile; r < ma.R; r += gridDim.y * gridDim.z) {
            periodic_root_wg<16>(g, r, ra.root_part, ra.box_part, ra.latT, ra.lat_seg, ra.root_m, ra.root_l, ra.dom,
                                 rt, rt + 2 * D::K, rt + D::K, blockDim.x);
            __syncthreads();
        }
        return;
    }
    const M2LTask tk = tasks[blockIdx.x];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int cg = wave / NRG, rg = wave - cg * NRG, kq = lane >> 4, row = lane & 15;
    const int cgs = blockDim.x / (64 * NRG);
    const int o0 = tk.o0, o1 = tk.o1;
    const int nthr = blockDim.x;
    auto issue = [&](int slot, uint4* dst) {
        const uint4* src = bank + ((size_t)slot * D::NPART + tk.tile) * D::a_chunks;
        for (int c0 = 64 * wave; c0 < D::a_chunks; c0 += nthr) lds_dma16(src + c0 + lane, dst + c0);
    };
    // the chunk's offsets, 64 at a time in a register (lane i: offset o0 + i)
    const int32_t* ol = olist + 189 * max(tk.cls, 0);
    int ol_reg = ol[min(o0 + lane, 188)];
    if (o0 < o1) issue(__builtin_amdgcn_readlane(ol_reg, 0) >> 16, op0);
    // this lane's column: replica, class, level and box
    const int u = (tile * cgs + cg) * 16 + row;
    const int per = ma.merged ? 8 * ma.ncol : ma.ncol;
    const int rep = u / per, rem = u - rep * per;
    const int cls = ma.merged ? rem / ma.ncol : tk.cls;
    int j = ma.merged ? rem - cls * ma.ncol : rem;
    const bool cok = rep < ma.R;
    const bool active = __ballot(cok) != 0;
    int lev = g.depth;
    while (lev > g.lmin && j >= 1 << (3 * (lev - 1))) {
        j -= 1 << (3 * (lev - 1));
        --lev;
    }
    const int sh = lev - 1, half = 1 << sh, n = 1 << lev;
    const int tx = 2 * (j >> (2 * sh)) + ((cls >> 2) & 1);
    const int ty = 2 * ((j >> sh) & (half - 1)) + ((cls >> 1) & 1);
    const int tz = 2 * (j & (half - 1)) + (cls & 1);
    const int fx = (cls & 4) ? -1 : 1, fy = (cls & 2) ? -1 : 1, fz = (cls & 1) ? -1 : 1;
    const T* mrow = mult_all + ((size_t)(cok ? rep : 0) * g.nbox + lev_offset(lev)) * g.Kp;
    const uint64_t* mk = masks + ((cok ? cls : 0) * 4 + kq) * 3;
    const uint64_t sg_tail = mk[1], sg_row = mk[2];
    uint64_t sg_src = mk[0];
    // source row of this lane's column at canonical offset oi (zeros: none)
    auto source = [&](int oi) -> const T* {
        int sx = tx - fx * (oi / 49 - 3), sy = ty - fy * ((oi / 7) % 7 - 3), sz = tz - fz * (oi % 7 - 3);
        bool ok = cok;
        if (g.periodic) {
            sx &= n - 1;
            sy &= n - 1;
            sz &= n - 1;
        } else {
            ok = ok & ((unsigned)sx < (unsigned)n) & ((unsigned)sy < (unsigned)n) & ((unsigned)sz < (unsigned)n);
        }
        return ok ? mrow + (size_t)morton(sx, sy, sz) * g.Kp : zrow;
    };
    // the pieces of one offset's source row that this lane multiplies
    struct Src {
        uint4 q[NF > 0 ? NF * (4 / E) : 1];
        T t[NT > 0 ? NT : 1];
    };
    constexpr int NQ = NF * (4 / E);  // whole pieces
    auto load_piece = [&](const T* src, Src& b, int i) {
        if (i < NQ) b.q[i] = *(const uint4*)(src + 4 * E * i + E * kq);
        else b.t[i - NQ] = src[min(16 * NF + 4 * (i - NQ) + kq, D::K - 1)];
    };
    using Acc = typename MmaAcc<T>::type;
    Acc acc[RTW];
#pragma unroll
    for (int t = 0; t < RTW; ++t) acc[t] = Acc{T(0), T(0), T(0), T(0)};
    Src b0, b1;
    if (active) {
        const T* s0 = o0 < o1 ? source(__builtin_amdgcn_readlane(ol_reg, 0) & 0xffff) : zrow;
#pragma unroll
        for (int i = 0; i < NQ + NT; ++i) load_piece(s0, b0, i);
    }
    const int arow = 16 * RTW * rg + row;
    auto step = [&](int oc, const uint4* A, uint4* nxt, const Src& cur, Src& next) {
        const int st = oc + 1 - o0;
        const bool more = oc + 1 < o1;
        if (more && (st & 63) == 0) ol_reg = ol[min(oc + 1 + lane, 188)];
        const int ent = __builtin_amdgcn_readlane(ol_reg, st & 63);
        __builtin_amdgcn_s_waitcnt(0);  // this lane's copies have landed
        __syncthreads();                // everyone's have; the other buffer is free
        if (more) issue(ent >> 16, nxt);
        if (!active) return;
        // the sign masks are formed at their use (hoisted out of the loop they
        // would take a register per coefficient)
        asm volatile("" : "+v"(sg_src));
        // the next chunk's operator fragments are read ahead where there are
        // registers for them (narrow FP64: read with the chunk)
        constexpr int AB = sizeof(T) == 4 || RTW == D::RTB ? 2 : 1;
        T a[AB][RTW][4], at[NT > 0 ? NT : 1][RTW];
        auto load_a = [&](int kc) {
#pragma unroll
            for (int t = 0; t < RTW; ++t)
#pragma unroll
                for (int h = 0; h < 4 / E; ++h) {
                    struct V { T v[E]; };
                    const V w = __builtin_bit_cast(V, A[((kc * 4 + kq) * (4 / E) + h) * RPB + arow + 16 * t]);
#pragma unroll
                    for (int e = 0; e < E; ++e) a[kc % AB][t][E * h + e] = w.v[e];
                }
        };
        auto load_at = [&]() {
            const T* At = (const T*)A + 16 * NF * RPB;
#pragma unroll
            for (int s = 0; s < NT; ++s)
#pragma unroll
                for (int t = 0; t < RTW; ++t) at[s][t] = At[(4 * s + kq) * RPB + arow + 16 * t];
        };
        if constexpr (NF > 0 && AB == 2) load_a(0);
        if constexpr (NF == 0) load_at();
        // the next offset's source rows are requested behind the first chunk's
        // products (the scheduling barriers keep them there, and the operator
        // reads of a chunk ahead of its products)
        auto load_next = [&]() {
            const T* ns = source(ent & 0xffff);
#pragma unroll
            for (int i = 0; i < NQ + NT; ++i) load_piece(ns, next, i);
        };
        if (NF == 0 && more) load_next();
#pragma unroll
        for (int kc = 0; kc < NF; ++kc) {
            if (AB == 1) load_a(kc);
            T b[4];
#pragma unroll
            for (int h = 0; h < 4 / E; ++h) {
                struct V { T v[E]; };
                const V w = __builtin_bit_cast(V, cur.q[kc * (4 / E) + h]);
#pragma unroll
                for (int e = 0; e < E; ++e) b[E * h + e] = flip(w.v[e], sg_src, 4 * kc + E * h + e);
            }
            if constexpr (sizeof(T) == 4) transpose_rows(b);
            if (AB == 2 && kc + 1 < NF) load_a(kc + 1);
            if (kc + 1 == NF) load_at();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int t = 0; t < RTW; ++t) acc[t] = mma4(a[kc % AB][t][s], b[s], acc[t]);
            __builtin_amdgcn_sched_barrier(0);
            if (kc == 0 && more) load_next();
        }
#pragma unroll
        for (int s = 0; s < NT; ++s) {
            // padding past K is never written: taken as zero
            const T b = 16 * NF + 4 * s + kq < D::K ? flip(cur.t[s], sg_tail, s) : T(0);
#pragma unroll
            for (int t = 0; t < RTW; ++t) acc[t] = mma4(at[s][t], b, acc[t]);
        }
    };
    Acc sum[kSeq ? 4 : 1][kSeq ? RTW : 1];
    int chunk = 0, ce = 0;  // the current chunk and its last offset + 1
    if constexpr (kSeq) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < RTW; ++t) sum[q][t] = Acc{T(0), T(0), T(0), T(0)};
        ce = 189 / ma.nchunk;
    }
    // the chunk that ends at offset oc goes to its sum
    auto fold = [&](int oc) {
        if constexpr (kSeq) {
            if (oc + 1 < ce) return;
            const int q = chunk < (ma.nchunk & ~3) ? chunk & 3 : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i)  // (an addend of 0 and no branch: the sums stay in registers)
#pragma unroll
                for (int t = 0; t < RTW; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) sum[i][t][v] += i == q ? acc[t][v] : T(0);
#pragma unroll
            for (int t = 0; t < RTW; ++t) acc[t] = Acc{T(0), T(0), T(0), T(0)};
            ++chunk;
            ce = (chunk + 1) * 189 / ma.nchunk;
        }
    };
    for (int oc = o0; oc < o1; oc += 2) {
        step(oc, op0, op1, b0, b1);
        fold(oc);
        if (oc + 1 < o1) {
            step(oc + 1, op1, op0, b1, b0);
            fold(oc + 1);
        }
    }
    if (!active || !cok) return;
    if constexpr (kSeq)
#pragma unroll
        for (int t = 0; t < RTW; ++t) acc[t] = (sum[0][t] + sum[1][t]) + (sum[2][t] + sum[3][t]);
    const int64_t box = lev_offset(lev) + morton(tx, ty, tz);
    T* dst = kSeq || ma.nchunk == 1 ? loc_all + ((size_t)rep * g.nbox + box) * g.Kp
                            : part_all + (((size_t)rep * ma.nchunk + tk.chunk) * ma.nt_all +
                                          (box - lev_offset(g.lmin))) * g.Kp;
#pragma unroll
    for (int t = 0; t < RTW; ++t) {
        const int rt = tk.tile * D::RTB + rg * RTW + t, r = 16 * rt + 4 * kq;
        if (r >= D::KP) break;
#pragma unroll
        for (int h = 0; h < 4 / E; ++h) {
            struct V { T v[E]; };
            V w;
#pragma unroll
            for (int e = 0; e < E; ++e) w.v[e] = flip((T)acc[t][E * h + e], sg_row, 4 * rt + E * h + e);
            *(uint4*)(dst + r + E * h) = __builtin_bit_cast(uint4, w);
        }
    }
}

}  // namespace fmmk
