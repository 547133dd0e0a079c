// k_gemm_wide.hip -- the fast path's projection for batches above 64 rows (and, from 17 rows, for
// unsplit outputs of few features).
//
// Y[M][N] = X[M][K] * W[N][K]^T with v_mfma_f32_16x16x32_bf16, M <= 256, K % 128 == 0.
// With one 16-feature tile per wave (k_gemm.hip) every wave reads the whole activation chunk
// from LDS for 16 features, and above 64 rows those reads, not the weight stream, set the
// time.  Here a block owns BM = 64 MT rows x BN = 16 NT WN features as 4 x WN waves of MT x NT
// tiles, so an operand read serves MT or NT MFMAs: with WN = 2 the LDS reads per k-step of 32
// are 8 (MT + NT) KiB for 8 MT NT MFMAs.  The rows may be split over blocks as well: a launch
// with few features fills the chip so without the traffic of split-K partial tiles.  Row blocks
// of one feature block are neighbours on one XCD, so the weights come from HBM once (6144 and 4096 x
// 4096 in two row blocks at 128 rows and four at 251: a launch fetches the weights' bytes, and
// the activations' once per XCD).
// Both operands go through LDS in chunks of 64 elements by direct-to-LDS loads, D stages in
// a ring (D - 1 chunks requested ahead).  A load moves 8 rows x 128 contiguous bytes; the
// 16-byte piece G of stage row r sits at slot 8 r + (G xor (r mod 8)), so the 16 rows that an MFMA
// operand reads at one G fall on distinct banks.  Each chunk is one barrier: past it every
// wave's loads of the chunk are in and every read of the chunk before is done, so the
// request for chunk c + D - 1 may overwrite it.  The compiler does not count direct-to-LDS loads
// when it places its waits, so operand reads, waits and the barrier are explicit.
// The order of a sum is that of k_gemm.hip: one accumulator per output and split, k in
// increasing order 32 at a time, split boundaries in 128-element units; so the matrix-core
// verifier's results do not depend on which of the two kernels a row count takes.
#include "mg_device.h"
#include "mg_kernels.h"

namespace mg {

typedef __bf16 bf16x8_w __attribute__((ext_vector_type(8)));
typedef float f32x4_w __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_w __attribute__((ext_vector_type(4)));

constexpr int WG_KC = 64;         // K per chunk
constexpr int WG_LDS = 160 * 1024;

template <int MT, int NT, int WN>
struct WideShape {
    static constexpr int NW = 4 * WN, BM = 64 * MT, BN = 16 * NT * WN;
    static constexpr int STAGE = (BM + BN) * WG_KC * 2;  // bytes
    static constexpr int D = WG_LDS / STAGE >= 4 ? 4 : 3;
    static_assert(D * STAGE <= WG_LDS, "the ring fits");
};

template <int N>
__device__ __forceinline__ void wg_wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
template <int N>
__device__ __forceinline__ void wg_wait_lgkm() {
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(N) : "memory");
}
template <int OFF>
__device__ __forceinline__ void wg_read(u32x4_w& v, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF));
}
// 64 x 16 bytes, lane i to slot i; AUX: cache policy
template <int AUX>
__device__ __forceinline__ void wg_load(const uint16_t* src, unsigned char* slots) {
    __builtin_amdgcn_global_load_lds(src, slots, 16, 0, AUX);
}
// names a fragment as read and written here (after a wait), so no use of it moves up
__device__ __forceinline__ void wg_touch(u32x4_w& v) { asm volatile("" : "+v"(v)); }

// the 16-row operand tiles I .. N - 1 of a k-step, 2 KiB apart
template <int N, int I = 0>
__device__ __forceinline__ void wg_read_tiles(u32x4_w (&v)[N], uint32_t addr) {
    if constexpr (I < N) {
        wg_read<I * 2048>(v[I], addr);
        wg_read_tiles<N, I + 1>(v, addr);
    }
}

template <int MT, int NT, int WN, int EPI>
__global__ __launch_bounds__(256 * WN, 2) void wide_gemm_kernel(FastGemmArgs a, int nfb, int nrb) {
    using S = WideShape<MT, NT, WN>;
    constexpr int NW = S::NW, BM = S::BM, BN = S::BN, D = S::D;
    static_assert(EPI != FEPI_SWIGLU || WN == 2, "gate and up waves");
    constexpr int LX = 2 * MT / WN;                  // activation loads per wave and chunk
    constexpr int LW0 = (NT + 1) / 2, LW1 = NT / 2;  // weight loads of the block's first and second half of waves
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int jl = lane & 15, q = lane >> 4;
    const int wm = wave / WN, wn = wave % WN;
    // blocks are dealt to the 8 XCDs round-robin: the row blocks of a feature block take
    // consecutive slots of one XCD
    const int slot = blockIdx.x >> 3, nb = slot / nrb * 8 + (blockIdx.x & 7), rb = slot % nrb;
    if (nb >= nfb) return;
    const int split = blockIdx.y, m0 = rb * BM;
    const int K = a.K, M = a.M;
    const bool lower = wave < NW / 2;

    __shared__ __attribute__((aligned(16))) unsigned char ring[D * S::STAGE];

    // this lane's piece of each of its wave's loads: load l covers stage rows 8 l .. 8 l + 7
    // (activation rows, then weight rows); rows past M and features past N re-read the last one
    const int lr = lane >> 3, lp = 8 * ((lane & 7) ^ lr);
    const uint16_t* xsrc[LX];
#pragma unroll
    for (int t = 0; t < LX; ++t) xsrc[t] = a.X + (size_t)min(m0 + 8 * (wave + NW * t) + lr, M - 1) * K + lp;
    const uint16_t* wsrc[LW0];
#pragma unroll
    for (int t = 0; t < LW0; ++t) {
        const int r = min(8 * (wave + NW * t), BN - 8) + lr;
        if constexpr (EPI == FEPI_SWIGLU) {
            // the block's first half of weight rows are gate rows, the others the same outputs' up rows
            const int up = r >= BN / 2, n = min(nb * (BN / 2) + r - up * (BN / 2), a.N - 1);
            wsrc[t] = a.W[up] + (size_t)n * K + lp;
        } else {
            int n = min(nb * BN + r, a.N - 1), seg = 0;
            while (seg < 2 && n >= a.Nseg[seg]) { n -= a.Nseg[seg]; ++seg; }
            wsrc[t] = a.W[seg] + (size_t)n * K + lp;
        }
    }
    // The weights are streamed ("nt") with several row blocks too: those run together and fetch no
    // more than with the default policy, which is 1 to 5% slower on the O and QKV shapes of 65 to
    // 256 rows.  The exception is a row block of 128 next to one at most half full, which runs ahead: 3 to 6%
    // of the weights are fetched again (4096 x 14336 at 192 rows 46 us, 43 with the default policy).
    auto issue = [&](int c, int stage) {
        unsigned char* buf = ring + stage * S::STAGE + 1024 * wave;
        const size_t k = (size_t)c * WG_KC;
#pragma unroll
        for (int t = 0; t < LX; ++t) wg_load<0>(xsrc[t] + k, buf + 1024 * NW * t);
#pragma unroll
        for (int t = 0; t < LW1; ++t) wg_load<MG_AUX_NT>(wsrc[t] + k, buf + BM * 128 + 1024 * NW * t);
        if (LW0 != LW1 && lower) wg_load<MG_AUX_NT>(wsrc[LW0 - 1] + k, buf + BM * 128 + 1024 * NW * (LW0 - 1));
    };

    const int nunits = K / 128;
    const int c0 = (int)((long)split * nunits / a.S) * (128 / WG_KC), c1 = (int)((long)(split + 1) * nunits / a.S) * (128 / WG_KC);

    f32x4_w acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4_w{0.f, 0.f, 0.f, 0.f};

    // operand addresses inside a stage: row jl of tile 0, k-step 0 (k-step 1 is 64 bytes away by xor)
    const uint32_t ring0 = (uint32_t)(uintptr_t)&ring[0];
    const uint32_t lane0 = jl * 128 + 16 * (q ^ (jl & 7));
    const uint32_t xl = lane0 + wm * MT * 2048, wl = lane0 + BM * 128 + wn * NT * 2048;

#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (c0 + d < c1) issue(c0 + d, d);
    int stage = 0;
    for (int c = c0; c < c1; ++c) {
        // this wave's loads of chunk c are in (D - 2 later chunks may be outstanding; near the end none)
        if (c + D - 2 >= c1) wg_wait_vmcnt<0>();
        else if (LW0 == LW1 || lower) wg_wait_vmcnt<(D - 2) * (LX + LW0)>();
        else wg_wait_vmcnt<(D - 2) * (LX + LW1)>();
        asm volatile("s_barrier" ::: "memory");
        const int back = stage == 0 ? D - 1 : stage - 1;
        if (c + D - 1 < c1) issue(c + D - 1, back);
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t sb = ring0 + stage * S::STAGE;
        u32x4_w xv[2][MT], wv[2][NT];
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const uint32_t xa = sb + (xl ^ (64 * st)), wa = sb + (wl ^ (64 * st));
            wg_read_tiles<NT>(wv[st], wa);
            wg_read_tiles<MT>(xv[st], xa);
        }
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            if (st == 0) wg_wait_lgkm<(MT + NT < 15 ? MT + NT : 15)>();
            else wg_wait_lgkm<0>();
#pragma unroll
            for (int i = 0; i < NT; ++i) wg_touch(wv[st][i]);
#pragma unroll
            for (int i = 0; i < MT; ++i) wg_touch(xv[st][i]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_w, xv[st][mt]),
                                                                          __builtin_bit_cast(bf16x8_w, wv[st][nt]), acc[mt][nt], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        stage = stage == D - 1 ? 0 : stage + 1;
    }

    // D[i][j] of a 16x16 tile sits in lane j + 16 (i / 4), element i % 4
    const int row0 = 16 * wm * MT + 4 * q;  // in the block's rows
    if constexpr (EPI == FEPI_SWIGLU) {
        // gate and up projections, rounded to bf16, meet in the ring (no load is outstanding); then
        // every thread takes 8 consecutive outputs of a row (the gate waves alone, 2 bytes a store, took
        // 9 us longer at 128 rows)
        constexpr int HN = 16 * NT, HS = HN + 8;  // outputs per row and block, and their LDS stride
        uint16_t* gu = reinterpret_cast<uint16_t*>(ring);  // [gate, up][BM][HS]
        static_assert(2 * BM * HS * 2 <= D * S::STAGE, "the bf16 tiles fit in the ring");
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    gu[(wn * BM + row0 + 16 * mt + v) * HS + 16 * nt + jl] = (uint16_t)f2bf(acc[mt][nt][v]);
        __syncthreads();
        uint16_t* act = reinterpret_cast<uint16_t*>(a.Y);
        for (int e = threadIdx.x; e < BM * (HN / 8); e += 64 * NW) {
            const int row = e / (HN / 8), n = e % (HN / 8) * 8;
            // (N % 16 == 0, so a group of 8 is inside the output or past it)
            if (m0 + row >= M || nb * HN + n >= a.N) continue;
            const uint4 g4 = *reinterpret_cast<const uint4*>(gu + row * HS + n);
            const uint4 u4 = *reinterpret_cast<const uint4*>(gu + (BM + row) * HS + n);
            const uint32_t gw[4] = {g4.x, g4.y, g4.z, g4.w}, uw[4] = {u4.x, u4.y, u4.z, u4.w};
            uint32_t o[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float g0 = bf_lo(gw[k]), g1 = bf_hi(gw[k]);
                o[k] = pack_bf2((g0 / (1.0f + __expf(-g0))) * bf_lo(uw[k]), (g1 / (1.0f + __expf(-g1))) * bf_hi(uw[k]));
            }
            *reinterpret_cast<uint4*>(act + (size_t)(m0 + row) * a.N + nb * HN + n) = make_uint4(o[0], o[1], o[2], o[3]);
        }
    } else if constexpr (EPI == FEPI_TOP2) {
        // per row: the top-2 of the wave's features, then of the row's waves (LDS)
        Top2* wst = reinterpret_cast<Top2*>(ring);  // [WN][BM]
        static_assert(WN * BM * (int)sizeof(Top2) <= D * S::STAGE, "the states fit in the ring");
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Top2 st{-__builtin_inff(), -__builtin_inff(), -1, 0};
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const int n = nb * BN + 16 * (wn * NT + nt) + jl;
                    if (n < a.N) top2_push(st, acc[mt][nt][v], n);
                }
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) st = top2_merge(st, top2_shfl(st, o));
                if (jl == 0)
                    *reinterpret_cast<uint4*>(&wst[wn * BM + row0 + 16 * mt + v]) =
                        make_uint4(__float_as_uint(st.v1), __float_as_uint(st.v2), (uint32_t)st.i1, (uint32_t)st.nan);
            }
        __syncthreads();
        for (int row = threadIdx.x; row < BM && m0 + row < M; row += 64 * NW) {
            auto ld = [&](int w) {
                const uint4 u = *reinterpret_cast<const uint4*>(&wst[w * BM + row]);
                return Top2{__uint_as_float(u.x), __uint_as_float(u.y), (int)u.z, (int)u.w};
            };
            const Top2 st = WN == 2 ? top2_merge(ld(0), ld(WN - 1)) : ld(0);
            reinterpret_cast<uint4*>(a.part)[(size_t)(m0 + row) * nfb + nb] =
                make_uint4(__float_as_uint(st.v1), __float_as_uint(st.v2), (uint32_t)st.i1, (uint32_t)st.nan);
        }
    } else {
        float* out = EPI == FEPI_F32 ? reinterpret_cast<float*>(a.Y) : a.part + (size_t)split * M * a.N;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int n = nb * BN + 16 * (wn * NT + nt) + jl;
            if (n >= a.N) continue;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = m0 + row0 + 16 * mt + v;
                    if (row < M) out[(size_t)row * a.N + n] = acc[mt][nt][v];
                }
        }
    }
}

bool wide_gemm_takes(int M, int K) { return M > 64 && M <= 256 && K % 128 == 0; }

struct WideLaunch {
    int MT, NT, WN;
    double cost;
};

// Estimated cycles of a launch.  Loads of the two operands do not overlap in a CU (gate/up
// at 128 rows: 71 us with both, 51 with the weights alone, 17 with the activations alone; a deeper
// ring changes nothing), so their times add: the activations, and the weights that another
// row block has already brought into the XCD's L2, at 32 bytes a cycle and CU; the other weights
// from HBM at 2375 bytes a cycle over the chip, at most 13 a CU.  LDS reads and MFMAs of a chunk
// take about 1.5 times the LDS port's time (4 WN (MT + NT) KiB read and 64 (BM + BN) bytes written
// per k-step of 32, 128 bytes a cycle).  4 us to start and end; split tiles are written and
// read once at about 2 KB a cycle.  The busiest CU is one of the XCD that gets the most blocks: the
// feature blocks are dealt to the XCDs whole, so 26 of them in 9 splits are 36 blocks for the 32
// CUs of two XCDs, a second round, though the chip has 256 CUs for 234 blocks (4096 x 14336 at 65
// rows 43 us so, 26 in 8 splits of 32 blocks an XCD; 3584 x 18944 at 128 rows 50 in 36 blocks an XCD,
// 35 in 27).  The tile that it takes for a split count is within 5% of the fastest one there for
// the QKV, O and down projections of the three models at 65..251 rows (all tiles measured one by
// one; 16% at 129 rows of 7168 x 5120); another split count would be up to a fifth faster where
// three or four splits of a down projection leave CUs idle (251 rows of 4096 x 14336: 58 us, 48 in 4).
static double wide_cost(int M, int N, int K, int MT, int NT, int WN, int S, int n_cu) {
    const int BM = 64 * MT, BN = 16 * NT * WN, nrb = (M + BM - 1) / BM;
    const long blocks = (long)(((N + BN - 1) / BN + 7) / 8) * nrb * S;  // of the XCD that has the most
    const long xcd_cu = n_cu >= 8 ? n_cu / 8 : 1;
    const long units = K / 128, ksteps = (units + S - 1) / S * 4;
    const double steps = (double)((blocks + xcd_cu - 1) / xcd_cu) * ksteps;  // k-steps of the busiest CU
    const double l2 = steps * 2.0 * (BM + BN * (1.0 - 1.0 / nrb));
    const double hbm_chip = (double)N * K * 2 / 2375.0, hbm_cu = steps * BN * 64.0 / nrb / 13.0;
    const double mem = l2 + (hbm_chip > hbm_cu ? hbm_chip : hbm_cu);
    const double chain = steps * 1.5 * (32.0 * WN * (MT + NT) + (BM + BN) / 2.0);
    return 9600.0 + (mem > chain ? mem : chain) + (S > 1 ? (double)S * M * N * 8 / 2083.0 : 0.0);
}

static WideLaunch wide_choose(int M, int N, int K, int S, bool pairs, int n_cu) {
    WideLaunch best{0, 0, 0, 0.0};
    const int mt_max = (M + 63) / 64;
    for (int MT = 1; MT <= mt_max; ++MT)
        for (int WN = 2; WN >= 1; --WN) {
            if (WN == 1 && (pairs || M > 128 || MT > 2)) continue;  // 4-wave blocks: no gate/up waves, up to 128 rows
            for (int NT = 1; NT <= (WN == 2 ? 5 : 3); ++NT) {
                const double c = wide_cost(M, N, K, MT, NT, WN, S, n_cu);
                if (!best.MT || c < best.cost) best = WideLaunch{MT, NT, WN, c};
            }
        }
    return best;
}

int wide_gemm_splits(int M, int N, int K, int S_max, int n_cu) {
    int best = 1;
    double bc = wide_choose(M, N, K, 1, false, n_cu).cost;
    for (int S = 2; S <= S_max; ++S) {
        const double c = wide_choose(M, N, K, S, false, n_cu).cost;
        if (c < bc) { bc = c; best = S; }
    }
    return best;
}

int wide_gemm_waves(int M, int N, int K, int S, int n_cu) { return 4 * wide_choose(M, N, K, S, false, n_cu).WN; }

int wide_gemm_blocks(int M, int N, int K, int n_cu) {
    const WideLaunch c = wide_choose(M, N, K, 1, false, n_cu);
    return (N + 16 * c.NT * c.WN - 1) / (16 * c.NT * c.WN);
}

template <int MT, int NT, int WN>
static void launch_wide_cfg(const FastGemmArgs& a, int epi, hipStream_t s) {
    const int per_block = (epi == FEPI_SWIGLU ? 8 : 16) * NT * WN;
    const int nfb = (a.N + per_block - 1) / per_block, nrb = (a.M + 64 * MT - 1) / (64 * MT);
    const dim3 g((nfb + 7) / 8 * 8 * nrb, a.S), b(256 * WN);
    switch (epi) {
        case FEPI_PART: hipLaunchKernelGGL((wide_gemm_kernel<MT, NT, WN, FEPI_PART>), g, b, 0, s, a, nfb, nrb); break;
        case FEPI_TOP2: hipLaunchKernelGGL((wide_gemm_kernel<MT, NT, WN, FEPI_TOP2>), g, b, 0, s, a, nfb, nrb); break;
        case FEPI_F32: hipLaunchKernelGGL((wide_gemm_kernel<MT, NT, WN, FEPI_F32>), g, b, 0, s, a, nfb, nrb); break;
        case FEPI_SWIGLU:
            if constexpr (WN == 2)  // (the choice for pairs)
                hipLaunchKernelGGL((wide_gemm_kernel<MT, NT, WN, FEPI_SWIGLU>), g, b, 0, s, a, nfb, nrb);
            break;
    }
}

template <int MT>
static void launch_wide_mt(const FastGemmArgs& a, int epi, const WideLaunch& c, hipStream_t s) {
    if constexpr (MT <= 2) {
        if (c.WN == 1) {
            if (c.NT == 1) return launch_wide_cfg<MT, 1, 1>(a, epi, s);
            if (c.NT == 2) return launch_wide_cfg<MT, 2, 1>(a, epi, s);
            return launch_wide_cfg<MT, 3, 1>(a, epi, s);
        }
    }
    switch (c.NT) {
        case 1: launch_wide_cfg<MT, 1, 2>(a, epi, s); break;
        case 2: launch_wide_cfg<MT, 2, 2>(a, epi, s); break;
        case 3: launch_wide_cfg<MT, 3, 2>(a, epi, s); break;
        case 4: launch_wide_cfg<MT, 4, 2>(a, epi, s); break;
        default: launch_wide_cfg<MT, 5, 2>(a, epi, s); break;
    }
}

hipError_t launch_wide_gemm(const FastGemmArgs& a, int epi, hipStream_t s) {
    if (a.M < 1 || a.M > 256 || a.K % 128) return hipErrorInvalidValue;
    if (epi != FEPI_PART && epi != FEPI_F32 && epi != FEPI_TOP2 && epi != FEPI_SWIGLU) return hipErrorInvalidValue;
    // a SwiGLU launch streams the gate and the up rows: 2N weight rows
    const bool pairs = epi == FEPI_SWIGLU;
    const WideLaunch c = wide_choose(a.M, pairs ? 2 * a.N : a.N, a.K, a.S, pairs, a.n_cu > 0 ? a.n_cu : 256);
    switch (c.MT) {
        case 1: launch_wide_mt<1>(a, epi, c, s); break;
        case 2: launch_wide_mt<2>(a, epi, c, s); break;
        case 3: launch_wide_mt<3>(a, epi, c, s); break;
        default: launch_wide_mt<4>(a, epi, c, s); break;
    }
    return hipGetLastError();
}

}  // namespace mg
