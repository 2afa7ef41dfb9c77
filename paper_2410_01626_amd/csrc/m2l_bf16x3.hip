// m2l_bf16x3.hip -- bf16x3 M2L on the matrix cores for trees whose classes have
// many target columns (depth >= 4, or orders whose resident-source form does
// not fit the LDS).
//
// The operator bank and the source expansions are stored pre-split into bf16
// hi/lo parts:
//   operator o: [part][KC][RP] chunks of 8 bf16 (chunk kc of row r holds
//               k = 8 kc .. 8 kc + 7), 2 KC RP chunks, zero padded;
//   boxes:      rows of one parity class in raster order, eight rows interleaved
//               in chunks (store_split): [row / 8][part][KC][row % 8].
// Products Th mh + Th ml + Tl mh accumulate in FP32 in the order of the offset
// list.  Every class works from the 189 operators of class 0 (the bank holds
// those in list order): reflecting the axes whose bit is set in the class maps
// class 0's offsets onto the class's own, and T(P o) = S T(o) S with S the
// diagonal +-1 reflection signs.  So a column of class c applies T(o') S of the
// canonical offset o' to mu of the source at offset P o', and its result is S
// times the accumulator (at the store).  The bank holds T(o') S for each class
// (k_sign_bank, at plan creation; signs on the source fragments instead took
// 160 vector instructions and as many register moves per offset).
//
// What bounds it: per offset a CU needs the 64 KB operator (p = 10) and one
// 512-byte source row per column, and multiplies for 16 cycles per 16 x 16 x 32
// product.  With 160 columns per work-group (four wavefronts: two row halves
// times two column halves of five 16-column groups) that is 3,840 cycles of
// products for 64 KB + 2 x 80 KB of loads, and the 4,681 columns a class has at
// depth 5 make 30 work-groups per class, one for each CU of the XCD that takes
// the class (its rows and the operator stream are then shared in that L2).
//  - Source rows go straight to registers (a lane's fragments are 16-byte
//    pieces of one row): the pieces of k-step s are reloaded for the next
//    offset as soon as this one's products have used them.
//  - The operator goes through registers into the other LDS buffer (one barrier
//    per offset; direct-to-LDS copies reach a third of the plain loads' rate).
//  - The sources of 16 neighbouring columns are neighbouring rows for every
//    offset (one shift of the halved coordinates), and eight rows interleaved
//    make a wavefront's load whole 128-byte lines: with a row per box, every
//    lane's 16 bytes cost an L1 lookup of their own and the kernel took 1,395 us.
// 500,000 atoms at depth 5, p = 10: 1,384 us (80 columns and one operator per
// work-group staged with global_load_lds in one LDS buffer) -> 630 us (986
// TFLOP/s of bf16 products; the products alone take about 350 us).

namespace fmmk {

constexpr int kBfThreads = 256;

// Class c's operators T(o') S from class 0's (copy 0 of the bank): sign bits of
// the input coefficients flipped.  One 16-byte chunk per thread.
__global__ __launch_bounds__(256) void k_sign_bank(uint4* __restrict__ bank, const uint4* __restrict__ sign_tab,
                                                   int64_t copy_chunks, int KC, int RP) {
    const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    const int c = blockIdx.y + 1;
    if (i >= copy_chunks) return;
    const uint4 m = sign_tab[c * 4 * kM2LMaxKs + (int)((i / RP) % KC)];
    uint4 v = bank[i];
    v.x ^= m.x;
    v.y ^= m.y;
    v.z ^= m.z;
    v.w ^= m.w;
    bank[c * copy_chunks + i] = v;
}

// Target columns of a work-group of CG column groups per wavefront.
__host__ __device__ constexpr int m2l_bf_cols(int rt, int cg) { return 16 * cg * (rt > 1 ? 2 : 4); }

template <int RT, int CG>
__global__ __launch_bounds__(kBfThreads) void k_m2l_bf16x3(Geo g, M2LGeom mg, const M2LTask* __restrict__ tasks,
                                                           const int16_t* __restrict__ olist,
                                                           const uint4* __restrict__ msplit,
                                                           const uint4* __restrict__ bank,
                                                           const uint4* __restrict__ sign_tab,
                                                           const uint4* __restrict__ zrow,
                                                           float* __restrict__ loc, float* __restrict__ part) {
    constexpr int KC = m2l_rs_kc(RT), NKS = KC / 4, RP = 16 * RT, a_chunks = 2 * KC * RP;
    constexpr int NRH = RT > 1 ? 2 : 1;           // row halves
    constexpr int RTW = (RT + NRH - 1) / NRH;     // row tiles of a wavefront
    constexpr int AL = (a_chunks + kBfThreads - 1) / kBfThreads;  // operator chunks of a thread
    constexpr int AH = (AL + 1) / 2;
    __shared__ uint4 op[2][a_chunks];
    const M2LTask tk = tasks[blockIdx.x];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int rh = wave % NRH, cp = wave / NRH, kq = lane >> 4, row = lane & 15;
    // first row tile (an odd count: the halves share the middle tile)
    const int rt0 = rh ? RT - RTW : 0;
    msplit += (size_t)blockIdx.y * (g.nbox + 1) * 2 * KC;
    loc += (size_t)blockIdx.y * g.nbox * g.Kp;
    if (part) part += (size_t)blockIdx.y * mg.nchunk * mg.nt_all * g.Kp;
    const int o0 = tk.o0, o1 = tk.o1;
    // the chunk's offsets in LDS (a load in the loop would have every row load
    // before it waited for)
    __shared__ int offs[189];
    if (tid < 189) offs[tid] = olist[tk.cls * 189 + tid];
    __syncthreads();
    // this lane's columns, in raster order of the halved coordinates u (deepest
    // level first): u, its level (0: past the class's last column, reads zeros)
    // (and the level's first row of the split array)
    int cu[CG], csh[CG];
    uint32_t crow[CG];
    bool cok[CG];
#pragma unroll
    for (int i = 0; i < CG; ++i) {
        int u = tk.tile * m2l_bf_cols(RT, CG) + (cp * CG + i) * 16 + row, lev = g.depth;
        cok[i] = u < mg.ncol;
        while (lev > g.lmin && u >= 1 << (3 * (lev - 1))) {
            u -= 1 << (3 * (lev - 1));
            --lev;
        }
        cu[i] = u;
        csh[i] = lev - 1;
        crow[i] = (uint32_t)(lev_offset(lev) - 1);
    }
    // source rows of this lane's columns at canonical offset oi: the boxes
    // 2 u + c - o of each axis are 2 (u + d) + q, one shift d and one parity q
    // for all columns
    auto sources = [&](int oi, const uint4* (&src)[CG]) {
        const int ax = ((tk.cls >> 2) & 1) - ((tk.cls & 4) ? -1 : 1) * (oi / 49 - 3);
        const int ay = ((tk.cls >> 1) & 1) - ((tk.cls & 2) ? -1 : 1) * ((oi / 7) % 7 - 3);
        const int az = (tk.cls & 1) - ((tk.cls & 1) ? -1 : 1) * (oi % 7 - 3);
        const int q = ((ax & 1) << 2) | ((ay & 1) << 1) | (az & 1);
#pragma unroll
        for (int i = 0; i < CG; ++i) {
            const int sh = csh[i], hm = (1 << sh) - 1;
            const int x = (cu[i] >> (2 * sh)) + (ax >> 1), y = ((cu[i] >> sh) & hm) + (ay >> 1), z = (cu[i] & hm) + (az >> 1);
            bool ok = cok[i];
            if (!g.periodic) ok = ok & (((x | y | z) & ~hm) == 0);
            const uint32_t r = crow[i] + (q << (3 * sh)) + (((((x & hm) << sh) + (y & hm)) << sh) | (z & hm));
            src[i] = (ok ? msplit + (size_t)(r >> 3) * (16 * KC) + (r & 7) : zrow) + 8 * kq;
        }
    };
    uint4 bh[NKS][CG], bl[NKS][CG];
    auto load_b = [&](const uint4* const (&src)[CG], int si) {
#pragma unroll
        for (int i = 0; i < CG; ++i) {
            bh[si][i] = src[i][32 * si];
            bl[si][i] = src[i][8 * KC + 32 * si];
        }
    };
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    // an operator passes through registers in two halves
    u4 ra[AH];
    bank += (size_t)tk.cls * 189 * a_chunks;
    auto load_a = [&](int oc, int h) {
        const u4* src = (const u4*)(bank + (size_t)oc * a_chunks);
#pragma unroll
        for (int i = 0; i < AH; ++i) ra[i] = src[min((h * AH + i) * kBfThreads + tid, a_chunks - 1)];
    };
    auto store_a = [&](uint4* dst, int h) {
#pragma unroll
        for (int i = 0; i < AH; ++i) {
            const int e = (h * AH + i) * kBfThreads;
            if (e + kBfThreads <= a_chunks || e + tid < a_chunks) ((u4*)dst)[e + tid] = ra[i];
        }
    };
    mf4 acc[CG][RTW];
#pragma unroll
    for (int i = 0; i < CG; ++i)
#pragma unroll
        for (int t = 0; t < RTW; ++t) acc[i][t] = mf4{0.f, 0.f, 0.f, 0.f};
    if (o0 < o1) {
        const uint4* src[CG];
        sources(__builtin_amdgcn_readfirstlane(offs[o0]), src);
#pragma unroll
        for (int si = 0; si < NKS; ++si) load_b(src, si);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            load_a(o0, h);
            store_a(op[0], h);
        }
    }
    __syncthreads();
    for (int oc = o0; oc < o1; ++oc) {
        const uint4* A = op[(oc - o0) & 1];
        uint4* nxt = op[(oc - o0 + 1) & 1];
        // the last offset asks for its own operands again (never used)
        const int nc = min(oc + 1, o1 - 1);
        const uint4* src[CG];
        sources(__builtin_amdgcn_readfirstlane(offs[nc]), src);
        load_a(nc, 0);
#pragma unroll
        for (int si = 0; si < NKS; ++si) {
            const int kc = 4 * si + kq;
            mbf8 ah[RTW], al[RTW];
#pragma unroll
            for (int t = 0; t < RTW; ++t) {
                ah[t] = __builtin_bit_cast(mbf8, A[kc * RP + 16 * (rt0 + t) + row]);
                al[t] = __builtin_bit_cast(mbf8, A[(KC + kc) * RP + 16 * (rt0 + t) + row]);
            }
#pragma unroll
            for (int i = 0; i < CG; ++i) {
                const mbf8 xh = __builtin_bit_cast(mbf8, bh[si][i]), xl = __builtin_bit_cast(mbf8, bl[si][i]);
#pragma unroll
                for (int t = 0; t < RTW; ++t) acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[t], xh, acc[i][t], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < RTW; ++t) acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[t], xl, acc[i][t], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < RTW; ++t) acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[t], xh, acc[i][t], 0, 0, 0);
            }
            load_b(src, si);
            // (the reloads stay behind this k-step's products and ahead of the
            // next one's)
            __builtin_amdgcn_sched_barrier(0);
            if (si == (NKS - 1) / 2) {
                store_a(nxt, 0);
                load_a(nc, 1);
            }
        }
        store_a(nxt, 1);
        __syncthreads();
    }
    // signs S on the output rows, stored straight from the accumulators: lane
    // (column, kq) holds rows 16 rt + 4 kq .. + 3 of its column
#pragma unroll
    for (int i = 0; i < CG; ++i) {
        if (!cok[i]) continue;
        const int sh = csh[i], hm = (1 << sh) - 1;
        const int64_t box = lev_offset(sh + 1) + morton(2 * (cu[i] >> (2 * sh)) + ((tk.cls >> 2) & 1),
                                                         2 * ((cu[i] >> sh) & hm) + ((tk.cls >> 1) & 1),
                                                         2 * (cu[i] & hm) + (tk.cls & 1));
        float* dst = mg.nchunk == 1
                         ? loc + (size_t)box * g.Kp
                         : part + ((size_t)tk.chunk * mg.nt_all + (box - lev_offset(g.lmin))) * g.Kp;
#pragma unroll
        for (int t = 0; t < RTW; ++t) {
            const int rt = rt0 + t;
            if (16 * rt + 4 * kq >= g.Kp) break;                 // padding rows past the stored row length
            if (NRH * RTW > RT && rh && t == 0) continue;        // the shared middle tile: the first half's
            const uint4 m = sign_tab[tk.cls * 4 * kM2LMaxKs + 2 * rt + (kq >> 1)];
            const uint32_t lo = (kq & 1) ? m.z : m.x, hi = (kq & 1) ? m.w : m.y;
            float4 o;
            o.x = ((lo >> 15) & 1u) ? -acc[i][t][0] : acc[i][t][0];
            o.y = ((lo >> 31) & 1u) ? -acc[i][t][1] : acc[i][t][1];
            o.z = ((hi >> 15) & 1u) ? -acc[i][t][2] : acc[i][t][2];
            o.w = ((hi >> 31) & 1u) ? -acc[i][t][3] : acc[i][t][3];
            *(float4*)(dst + 16 * rt + 4 * kq) = o;
        }
    }
}

}  // namespace fmmk
