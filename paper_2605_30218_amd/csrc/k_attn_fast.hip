// k_attn_fast.hip -- the fast path's decode attention, fused with the split-K sum of
// the QKV projection, the bias, RoPE and the tentative K/V append.
//
// One block of 4 waves per (row, KV head, position split), with all G query heads of the KV
// head, so that every K/V page is read once.  With one split (enough rows to fill the device)
// the block merges everything itself; with several (split-KV, for long contexts at small
// batch) split k takes an equal share of the pages of positions 0..p-1, split 0 also takes
// position p, and a second launch merges the splits' (m, l, O) in split order.
// Prologue: sums the QKV split partials of the block's features (the G query heads of
// the group, then k, then v) in split order, adds the bias and rounds to bf16 (the
// projection's rounding point); rotates q and k (rotate-half RoPE from the fp32
// cos/sin table, products and sums rounded separately, then bf16); appends K' and V
// to the paged cache at the row's position p (the tentative column) -- or, for the
// matrix-core verifier, to the row's own column buffer, leaving the cache untouched;
// keeps q' (bf16, the MFMA B operand) and k'_p, v_p in LDS, and copies the row's page indices
// for positions < p into LDS.  The wave's first K/V step is requested before any of that.
// Main loop: wave w takes the 32-position steps (page pairs) w, w + 4, ... of positions
// 0..p-1, both products on MFMA:
//   S[pos][c] = K[pos][:] . Q[c][:]   two 16-position tiles, K straight from the page as the A
//       operand, columns c = 0 .. NS G - 1 holding query head c mod G (copied NS times);
//   softmax online in the exp2 domain on the fp32 scores: lane c + 16 q holds column c's
//       positions 4 q .. 4 q + 3 of both tiles, so a row maximum is two shuffles;
//   O[c][d] += P[c][pos] V[pos][d]    with the 8 k indices of lane group q standing for the
//       positions its lanes hold, so that P goes from the scores' layout into the A operand
//       without leaving its lane.  V's B operand pairs two positions of one d: a lane loads 8
//       rows of V (8 consecutive d each) and pairs them with one v_perm per operand word.
// The probabilities stay 32-bit values: a probability is the exact sum of three bf16 terms
// (its leading, middle and last 8 significant bits), every product of a term with a bf16 V is
// exact, and MFMA accumulates in fp32.  Up to 5 heads the three terms are the NS = 3 copies of
// the columns (rows of the P operand, otherwise idle); for 6 to 8 heads NS = 2 copies carry the
// first two terms and a second MFMA adds the third.
// What bounds it: the K/V stream.  The vector-ALU P V product of the kernel before this one
// (8 fma and a shuffle per head and position group, two blocks per KV head above 4 heads) took
// about as long as the stream itself.  Per layer, before and after: 128 rows of 128..2048
// positions, 8 KV heads of 5 query heads, 167 and 105 us (5.4 TB/s); 251 rows of 40..700
// positions, 4 of 7, 78 and 48; 64 rows of 512..768, 8 of 4, 41 and 34 (4.9 TB/s); 9 rows of
// 4096..16384, with the merge, 96 and 82; one row of 512, 19 (with its merge) and 11.  The steady
// stream runs at 5.5 TB/s (6.1: a plain read); 8 us of each launch are its dependent first loads
// (position, page, K/V) and the merge.
// Epilogue: each wave's (m, l, O) goes to LDS; position p contributes its own partial
// (m = score of q' . k'_p, l = 1, O = v_p) in split 0; the partials are merged and
// out = bf16(O / L), or the split's merged partial is stored for the split merge.  Every
// split recomputes the prologue (q' is needed by all); only split 0 writes the column.
// The summation order depends on the context length and the split of positions over
// waves: this path is not the verifier's order.
#include <type_traits>

#include "mg_device.h"
#include "mg_kernels.h"

namespace mg {

typedef __bf16 bf16x8_ft __attribute__((ext_vector_type(8)));
typedef float f32x4_ft __attribute__((ext_vector_type(4)));

#ifndef MG_FA_MIN_WAVES
#define MG_FA_MIN_WAVES 3  // waves per SIMD the register budget must allow (three blocks per CU)
#endif
constexpr int FA_WAVES = 4;
constexpr int FA_THREADS = 64 * FA_WAVES;
constexpr int FA_PGCAP = 1024;  // page indices held in LDS (positions < 16384); more are read from memory
constexpr int FA_MAXB = 256;    // rows of a step

__device__ __forceinline__ float fa_scale(int hd) { return hd == 128 ? 0x1.6a09e6p-4f : 0x1.0p-3f; }

// two fp32 values whose lower 16 bits are dropped, as a bf16 pair
__device__ __forceinline__ uint32_t top_halves(float lo, float hi) {
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
// NW words of the K/V stream, with the "nt" policy where NTP
template <class T, int NW, bool NTP>
__device__ __forceinline__ T kv_load(const uint16_t* p) {
    using v = uint32_t __attribute__((ext_vector_type(NW)));
    const v* q = reinterpret_cast<const v*>(p);
    return __builtin_bit_cast(T, NTP ? __builtin_nontemporal_load(q) : *q);
}
__device__ __forceinline__ float cut_bf16(float x) { return __uint_as_float(__float_as_uint(x) & 0xffff0000u); }

template <int HD, int G, bool NTP>  // G: query heads per KV head, 1..8; NTP: cache policy of the K/V loads
__global__ __launch_bounds__(FA_THREADS) __attribute__((amdgpu_waves_per_eu(MG_FA_MIN_WAVES))) void attn_fast_fused_kernel(FastAttnArgs a) {
    constexpr int KST = HD / 32;         // MFMA k-steps over d
    constexpr int H2 = HD / 2;
    constexpr int VD = HD / 16;          // consecutive d per lane of a V row: MFMA tile t holds d = VD jl + t
    constexpr int VW = VD / 2;           // words of them
    constexpr int NS = G <= 5 ? 3 : 2;   // copies of the head columns (bf16 terms of P)
    constexpr int NC = NS * G;           // live columns
    static_assert(NC <= 16, "columns of one MFMA tile");
    const ModelDims& m = a.m;
    const int Nq = m.Hq * HD, Nk = m.Hkv * HD, N = Nq + 2 * Nk;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int jl = lane & 15, qg = lane >> 4;
    const float sl2 = fa_scale(HD) * 1.4426950408889634f;  // scores in log2 units

    __shared__ float y[(G + 2) * HD];
    __shared__ __attribute__((aligned(16))) uint16_t qb[G * HD];
    __shared__ float kps[HD], vps[HD];
    __shared__ int pgs[FA_PGCAP];
    __shared__ float sp[G];
    __shared__ float wm[FA_WAVES][G], wl[FA_WAVES][G];
    __shared__ __attribute__((aligned(16))) float wo[FA_WAVES][NC][HD];

    const int kh = blockIdx.x % m.Hkv, split = blockIdx.z;
    int r = blockIdx.x / m.Hkv, p;
    if (a.longest_first) {
        // blocks are dispatched in index order: block index u / Hkv takes the row whose context
        // is the (u / Hkv)-th longest (ties by row), so that no long row starts when the others
        // are nearly done.  Every wave finds it from all rows' positions, row 64 k + lane in pos[k]:
        // the position bit by bit from the count of rows at or above a candidate, then the row
        // among those at that position, some 12 counts of 4 ballots.  (Each thread counting the rows
        // before its own took all rows' compares on the vector ALUs in every block: two layers of 251
        // rows at 40..700 positions and 4 KV heads 507 us with their projections, 485 so; of 200 rows at
        // up to 100 positions and 8 KV heads 201 and 171.)
        constexpr int NP = FA_MAXB / 64;
        int pos[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) pos[k] = 64 * k + lane < a.B ? a.positions[64 * k + lane] : -1;
        p = 0;
        for (int bit = 31 - __builtin_clz(16 * m.max_pages_per_row); bit >= 0; --bit) {
            const int cand = p | (1 << bit);
            int cnt = 0;
#pragma unroll
            for (int k = 0; k < NP; ++k) cnt += __popcll(__ballot(pos[k] >= cand));
            if (cnt > r) p = cand;
        }
        int n = r;  // the row's place among those at position p
#pragma unroll
        for (int k = 0; k < NP; ++k) n -= __popcll(__ballot(pos[k] > p));
        r = 0;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const unsigned long long at = __ballot(pos[k] == p);
            const int c = __popcll(at);
            if (n >= 0 && n < c) {
                const bool me = ((at >> lane) & 1) && __popcll(at & ((1ull << lane) - 1)) == n;
                r = 64 * k + __ffsll(__ballot(me)) - 1;
            }
            n -= c;
        }
    } else {
        p = a.positions[r];
    }
    const int32_t* ptab = a.page_table + (size_t)r * m.max_pages_per_row;
    const int npg = (p + 15) / 16;  // pages holding positions 0..p-1
    // this split's pages [pg0, pg1): a fixed share of the capacity, so a block's work is
    // bounded whatever the row's length; a split past the row's pages has nothing to do (the
    // merge reads only the row's live splits)
    const int pg0 = split * a.split_pages, pg1 = min(npg, pg0 + a.split_pages);
    const bool first = split == 0;
    if (!first && pg0 >= npg) return;
    const bool pg_lds = pg1 - pg0 <= FA_PGCAP;
    const int lim = min(p, 16 * pg1);  // positions of this split: 16 pg0 .. lim - 1
    const int nst = (pg1 - pg0 + 1) / 2;  // its 32-position steps

    // loads of step s (positions 32 s .. 32 s + 31 from 16 pg0; pages pa, pb): K rows straight
    // into A-operand registers; V rows 4 qg .. 4 qg + 3 of both pages, this lane's VD values of d.
    // A last page past the split re-reads the one before it: its scores are masked and its V zeroed.
    using vload_t = typename std::conditional<VW == 4, uint4, uint2>::type;
    const size_t kv_stride = (size_t)m.Hkv * 16 * HD;  // K -> V of the same page
    const uint16_t* layer_kv = a.kv_pool + (((size_t)a.layer * m.n_pages * 2) * m.Hkv + kh) * (size_t)16 * HD;
    auto fetch_k = [&](int pa, int pb, uint4 (&kb)[2][KST]) {
        const uint16_t* kp[2] = {layer_kv + (size_t)pa * 2 * kv_stride, layer_kv + (size_t)pb * 2 * kv_stride};
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int st = 0; st < KST; ++st)
                kb[u][st] = kv_load<uint4, 4, NTP>(kp[u] + jl * HD + st * 32 + qg * 8);
    };
    auto fetch_v = [&](int pa, int pb, vload_t (&vb)[8]) {
        const uint16_t* vp[2] = {layer_kv + (size_t)pa * 2 * kv_stride + kv_stride,
                                 layer_kv + (size_t)pb * 2 * kv_stride + kv_stride};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            vb[i] = kv_load<vload_t, VW, NTP>(vp[i >> 2] + (4 * qg + (i & 3)) * HD + VD * jl);
    };
    auto pages_of = [&](int s, int& pa, int& pb) {
        const int ia = pg0 + 2 * s, ib = min(ia + 1, pg1 - 1);
        if (pg_lds) {
            pa = __builtin_amdgcn_readfirstlane(pgs[ia - pg0]);
            pb = __builtin_amdgcn_readfirstlane(pgs[ib - pg0]);
        } else {
            pa = ptab[ia];
            pb = ptab[ib];
        }
    };

    // ---- prologue.  Everything it reads is requested before any of it is used: the wave's first
    // page indices, the page table, the cos/sin pair, the first eight split partials, then (loads
    // complete in order) the first K/V step, whose latency passes under the rest
    constexpr int nf = (G + 2) * HD;                                // features: q heads, k, v
    constexpr int IT = (nf / 4 + FA_THREADS - 1) / FA_THREADS;      // groups of 4 per thread
    constexpr int PB = 8;                                           // split partials per batch
    uint4 kb[2][KST];
    vload_t vb[8];
    {
        const int last = max(pg1 - 1, 0);
        const int pa = ptab[min(pg0 + 2 * wave, last)], pb = ptab[min(pg0 + 2 * wave + 1, last)];
        const int own_page = ptab[p / 16];
        const int pgv = ptab[min(pg0 + t, last)];
        // (H2 divides the block: a thread's rotation pairs all have the same frequency)
        const float2 cs2 = *reinterpret_cast<const float2*>(a.cs + (size_t)p * HD + 2 * (t % H2));
        // split sum + bias + bf16 of this block's q, k, v features, the splits in split order
        const float* pp = a.part + (size_t)r * N;
        const size_t sstride = (size_t)a.B * N;
        int n[IT];
        float4 u[IT][PB];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int f = 4 * min(t + FA_THREADS * it, nf / 4 - 1);
            n[it] = f < G * HD ? kh * G * HD + f : f < (G + 1) * HD ? Nq + kh * HD + f - G * HD
                                                                    : Nq + Nk + kh * HD + f - (G + 1) * HD;
#pragma unroll
            for (int k = 0; k < PB; ++k)
                u[it][k] = k < a.S ? *reinterpret_cast<const float4*>(pp + (size_t)k * sstride + n[it])
                                   : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (wave < nst) {
            fetch_k(pa, pb, kb);
            fetch_v(pa, pb, vb);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (pg_lds) {
            if (t < pg1 - pg0) pgs[t] = pgv;
            for (int j = t + FA_THREADS; j < pg1 - pg0; j += FA_THREADS) pgs[j] = ptab[pg0 + j];
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int f = 4 * (t + FA_THREADS * it);
            float4 v = u[it][0];
#pragma unroll
            for (int k = 1; k < PB; ++k)
                if (k < a.S) { v.x += u[it][k].x; v.y += u[it][k].y; v.z += u[it][k].z; v.w += u[it][k].w; }
            for (int k = PB; k < a.S; ++k) {
                const float4 w = *reinterpret_cast<const float4*>(pp + (size_t)k * sstride + n[it]);
                v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
            }
            if (a.bq) {
                const uint16_t* b = f < G * HD ? a.bq + n[it] : f < (G + 1) * HD ? a.bk + n[it] - Nq : a.bv + n[it] - Nq - Nk;
                v.x += bf2f(b[0]); v.y += bf2f(b[1]); v.z += bf2f(b[2]); v.w += bf2f(b[3]);
            }
            if (f < nf) {
                y[f] = bf2f(f2bf(v.x));
                y[f + 1] = bf2f(f2bf(v.y));
                y[f + 2] = bf2f(f2bf(v.z));
                y[f + 3] = bf2f(f2bf(v.w));
            }
        }
        __syncthreads();
        // RoPE on q and k, tentative K/V append at p, q' / k'_p / v_p into LDS.  The tentative
        // column goes into the cache, or (own_out) the row's own column buffer
        uint16_t* kdst = a.own_out ? a.own_out + ((size_t)r * m.L + a.layer) * 2 * Nk + (size_t)kh * HD
                                   : const_cast<uint16_t*>(layer_kv) + (size_t)own_page * 2 * kv_stride + (size_t)(p % 16) * HD;
        uint16_t* vdst = kdst + (a.own_out ? (size_t)Nk : kv_stride);
        static_assert(FA_THREADS % H2 == 0, "one frequency per thread");
        for (int t2 = t; t2 < (G + 1) * H2; t2 += FA_THREADS) {
            const int head = t2 / H2, ii = t2 % H2;  // head == G: the k head
            const float* s = y + head * HD;
            const float x1 = s[ii], x2 = s[ii + H2];
            const float c = cs2.x, sn = cs2.y;
            const float ac = x1 * c, bs = x2 * sn, bc = x2 * c, as = x1 * sn;
            const uint32_t o1 = f2bf(ac - bs), o2 = f2bf(bc + as);
            if (head < G) {
                qb[head * HD + ii] = (uint16_t)o1;
                qb[head * HD + ii + H2] = (uint16_t)o2;
            } else {
                if (first) {
                    kdst[ii] = (uint16_t)o1;
                    kdst[ii + H2] = (uint16_t)o2;
                }
                kps[ii] = bf2f(o1);
                kps[ii + H2] = bf2f(o2);
            }
        }
        for (int d = t; d < HD; d += FA_THREADS) {
            const float v = y[(G + 1) * HD + d];
            if (first) vdst[d] = (uint16_t)f2bf(v);
            vps[d] = v;
        }
    }
    __syncthreads();

    // ---- position p's own score (log2 units): wave w takes heads w, w + 4
#pragma unroll
    for (int hh = 0; hh < (G + FA_WAVES - 1) / FA_WAVES; ++hh) {
        const int h = wave + FA_WAVES * hh;
        if (h < G) {
            float s = 0.0f;
            for (int d = lane; d < HD; d += 64) s += bf2f(qb[h * HD + d]) * kps[d];
            s = wave_sum_fast(s);
            if (lane == 0) sp[h] = s * sl2;
        }
    }

    // ---- main loop over this split's positions
    const int term = jl / G;  // which bf16 term of P this lane's column carries
    uint4 qa[KST];
#pragma unroll
    for (int st = 0; st < KST; ++st)
        qa[st] = jl < NC ? *reinterpret_cast<const uint4*>(qb + (jl % G) * HD + st * 32 + qg * 8) : make_uint4(0, 0, 0, 0);
    float mrun = -__builtin_inff(), lrun = 0.0f;  // of column jl; l over this lane's positions
    f32x4_ft o[VD];                               // O[4 qg + v][VD jl + tt]
#pragma unroll
    for (int tt = 0; tt < VD; ++tt) o[tt] = f32x4_ft{0.f, 0.f, 0.f, 0.f};

    // One step: the scores; then the wave's next K step is requested into the registers the
    // scores have used up, and after P V its next V step likewise.  A wave has a K or a V step in
    // flight at all times and three blocks share a CU; a second buffer of each would halve that
    // and spill
    for (int s = wave; s < nst; s += FA_WAVES) {
        const int base = 16 * pg0 + 32 * s;
        const bool more = s + FA_WAVES < nst;
        int pa = 0, pb = 0;
        if (more) pages_of(s + FA_WAVES, pa, pb);
        f32x4_ft sc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            sc[u] = f32x4_ft{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < KST; ++st)
                sc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_ft, kb[u][st]),
                                                                __builtin_bit_cast(bf16x8_ft, qa[st]), sc[u], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) fetch_k(pa, pb, kb);
        __builtin_amdgcn_sched_barrier(0);
        float x[8];  // positions base + 16 (i / 4) + 4 qg + i % 4 of column jl
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = sc[i >> 2][i & 3] * sl2;
        if (base + 32 > lim) {  // the last step: positions past the split are masked, their V zeroed
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const bool live = base + 16 * (i >> 2) + 4 * qg + (i & 3) < lim;
                x[i] = live ? x[i] : -__builtin_inff();
                uint32_t* w = reinterpret_cast<uint32_t*>(&vb[i]);
#pragma unroll
                for (int k = 0; k < VW; ++k) w[k] = live ? w[k] : 0u;
            }
        }
        float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(mrun, mx);
        const float alpha = exp2f(mrun - mn);
        mrun = mn;
        float psum = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            x[i] = exp2f(x[i] - mn);
            psum += x[i];
        }
        lrun = lrun * alpha + psum;
        if (__any(alpha != 1.0f)) {  // (a NaN counts) rescale: row 4 qg + v's factor sits in lane 4 qg + v
            float al[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) al[v] = __shfl(alpha, 4 * qg + v, 64);
#pragma unroll
            for (int tt = 0; tt < VD; ++tt)
#pragma unroll
                for (int v = 0; v < 4; ++v) o[tt][v] *= al[v];
        }
        // this column's term of P: the leading 8 significant bits, the next 8, the last 8
        uint4 pw, pl;
        {
            float w1[8], w2[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float r1 = x[i] - cut_bf16(x[i]), r2 = r1 - cut_bf16(r1);
                w1[i] = jl >= NC ? 0.0f : term == 0 ? x[i] : term == 1 ? r1 : r2;
                w2[i] = jl < G ? r2 : 0.0f;
            }
            pw = make_uint4(top_halves(w1[0], w1[1]), top_halves(w1[2], w1[3]), top_halves(w1[4], w1[5]),
                            top_halves(w1[6], w1[7]));
            pl = make_uint4(top_halves(w2[0], w2[1]), top_halves(w2[2], w2[3]), top_halves(w2[4], w2[5]),
                            top_halves(w2[6], w2[7]));
        }
        const bf16x8_ft PA = __builtin_bit_cast(bf16x8_ft, pw), PL = __builtin_bit_cast(bf16x8_ft, pl);
#pragma unroll
        for (int tt = 0; tt < VD; ++tt) {
            const uint32_t sel = (tt & 1) ? 0x07060302u : 0x05040100u;
            uint32_t w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                w[k] = __builtin_amdgcn_perm(reinterpret_cast<const uint32_t*>(&vb[2 * k + 1])[tt >> 1],
                                             reinterpret_cast<const uint32_t*>(&vb[2 * k])[tt >> 1], sel);
            const bf16x8_ft VB = __builtin_bit_cast(bf16x8_ft, make_uint4(w[0], w[1], w[2], w[3]));
            o[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(PA, VB, o[tt], 0, 0, 0);
            if constexpr (NS == 2) o[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(PL, VB, o[tt], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) fetch_v(pa, pb, vb);
    }

    // ---- wave partials: l over the lane groups; O's rows as they are (summed over the terms below)
    lrun += __shfl_xor(lrun, 16, 64);
    lrun += __shfl_xor(lrun, 32, 64);
    if (lane < G) {
        wm[wave][lane] = mrun;
        wl[wave][lane] = lrun;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (4 * qg + v < NC) {
            float* dst = &wo[wave][4 * qg + v][VD * jl];
#pragma unroll
            for (int tt = 0; tt < VD; tt += 4)
                *reinterpret_cast<float4*>(dst + tt) = make_float4(o[tt][v], o[tt + 1][v], o[tt + 2][v], o[tt + 3][v]);
        }
    }
    __syncthreads();

    // ---- merge the wave partials and (split 0) position p
    for (int oi = t; oi < G * HD; oi += FA_THREADS) {
        const int h = oi / HD, d = oi % HD;
        float M = first ? sp[h] : -__builtin_inff();
#pragma unroll
        for (int w = 0; w < FA_WAVES; ++w) M = fmaxf(M, wm[w][h]);
        float L = 0.0f, O = 0.0f;
        if (first) {
            const float ws = exp2f(sp[h] - M);
            L = ws;
            O = ws * vps[d];
        }
        if (M != -__builtin_inff()) {  // (a split with no position keeps L = O = 0)
#pragma unroll
            for (int w = 0; w < FA_WAVES; ++w) {
                const float ww = exp2f(wm[w][h] - M);
                float ov = wo[w][h][d];
                if constexpr (NS == 3) ov += wo[w][G + h][d] + wo[w][2 * G + h][d];
                else ov += wo[w][G + h][d];
                L += ww * wl[w][h];
                O += ww * ov;
            }
        }
        if (a.nsplit == 1) {
            a.out[(size_t)r * Nq + (size_t)(kh * G + h) * HD + d] = (uint16_t)f2bf(O / L);
        } else {
            float* dst = a.split_part + (((size_t)r * m.Hq + kh * G + h) * a.nsplit + split) * (HD + 2);
            if (d == 0) {
                dst[0] = M;
                dst[1] = L;
            }
            dst[2 + d] = O;
        }
    }
}

// The split merge of split-KV: for each (row, query head), the splits' (m, l, O) combined in
// split order (exp2 domain, as the partials), out = bf16(O / L).
__global__ void attn_fast_split_merge_kernel(FastAttnArgs a) {
    const int h = blockIdx.x, r = blockIdx.y, d = threadIdx.x;
    const int hd = a.m.hd, ns = a.nsplit;
    if (d >= hd) return;
    // the row's live splits: split 0 (position p) and those holding pages of positions < p
    const int npg = (a.positions[r] + 15) / 16;
    const int live = max(1, min(ns, (npg + a.split_pages - 1) / a.split_pages));
    const float* base = a.split_part + ((size_t)r * a.m.Hq + h) * ns * (hd + 2);
    // batches of 8 splits, every load of a batch in flight together (one split after the other,
    // each waiting for the one before, took 12.5 us at 9 rows of 17 splits)
    constexpr int MB = 8;
    float M = -__builtin_inff(), L = 0.0f, O = 0.0f;
    for (int k0 = 0; k0 < live; k0 += MB) {
        float mk[MB], lk[MB], ok[MB];
#pragma unroll
        for (int k = 0; k < MB; ++k) {
            const float* pk = base + (size_t)min(k0 + k, live - 1) * (hd + 2);
            mk[k] = pk[0];
            lk[k] = pk[1];
            ok[k] = pk[2 + d];
        }
        float mn = M;
#pragma unroll
        for (int k = 0; k < MB; ++k) mn = fmaxf(mn, mk[k]);
        if (mn == -__builtin_inff()) continue;  // no position so far
        const float w0 = exp2f(M - mn);
        M = mn;
        L *= w0;
        O *= w0;
#pragma unroll
        for (int k = 0; k < MB; ++k) {
            if (k0 + k >= live || mk[k] == -__builtin_inff()) continue;  // a split with no position
            const float w = exp2f(mk[k] - mn);
            L += w * lk[k];
            O += w * ok[k];
        }
    }
    a.out[(size_t)r * a.m.Hq * hd + (size_t)h * hd + d] = (uint16_t)f2bf(O / L);
}

template <int HD, int G>
static void launch_g(const FastAttnArgs& a, dim3 grid, bool stream, hipStream_t s) {
    if (stream)
        hipLaunchKernelGGL((attn_fast_fused_kernel<HD, G, true>), grid, dim3(FA_THREADS), 0, s, a);
    else
        hipLaunchKernelGGL((attn_fast_fused_kernel<HD, G, false>), grid, dim3(FA_THREADS), 0, s, a);
}

template <int HD>
static void launch_hd(const FastAttnArgs& a, int G, dim3 grid, bool stream, hipStream_t s) {
    switch (G) {
        case 1: launch_g<HD, 1>(a, grid, stream, s); break;
        case 2: launch_g<HD, 2>(a, grid, stream, s); break;
        case 3: launch_g<HD, 3>(a, grid, stream, s); break;
        case 4: launch_g<HD, 4>(a, grid, stream, s); break;
        case 5: launch_g<HD, 5>(a, grid, stream, s); break;
        case 6: launch_g<HD, 6>(a, grid, stream, s); break;
        case 7: launch_g<HD, 7>(a, grid, stream, s); break;
        default: launch_g<HD, 8>(a, grid, stream, s); break;
    }
}

hipError_t launch_fast_attention(const FastAttnArgs& args, hipStream_t s) {
    FastAttnArgs a = args;
    if (a.B <= 0) return hipSuccess;
    const int G = a.m.Hq / a.m.Hkv;
    if (G < 1 || G > 8 || a.B > FA_MAXB || a.m.page_size != 16 || (a.m.hd != 64 && a.m.hd != 128))
        return hipErrorInvalidValue;
    if (a.nsplit < 1 || a.split_pages < 1 || (long)a.nsplit * a.split_pages < a.m.max_pages_per_row ||
        (a.nsplit > 1 && !a.split_part))
        return hipErrorInvalidValue;
    // more blocks than two per CU: the longest rows first, where rows can differ by more than finding
    // them costs (two layers of 128 rows, 8 KV heads of 4 query heads, contexts of half to all of 2200
    // positions 396 against 428 us in the rows' own order, of 500 179 against 182, but of 300 159
    // against 154)
    const int units = a.B * a.m.Hkv;
    a.longest_first = a.nsplit == 1 && units > 2 * (a.n_cu > 0 ? a.n_cu : 256) && a.m.max_pages_per_row >= 32;
    const dim3 grid(units, 1, a.nsplit);
    // Launches of a block per CU and more are bound by the K/V stream, which then goes past the
    // caches' replacement ("nt": 128 rows of 128..2048 positions 108 us a layer against 121 with the default
    // policy, 4 us of each for an earlier row search; 64 rows of 512..768 34 against 36); smaller ones wait for single loads, which
    // the caches may still hold (one row of 512 positions: 13.9 against 13.0).  Pages that rows
    // share are read by each row's blocks, from the caches if they are kept there: a two-layer step of 32
    // or 64 rows on one prefix of 512 to 4096 positions is 3 to 5% slower with the policy, of
    // 128 rows on 1024 2% faster; which pages are shared stands in device memory only
    const bool stream = (long)units * a.nsplit >= (a.n_cu > 0 ? a.n_cu : 256);
    if (a.m.hd == 128)
        launch_hd<128>(a, G, grid, stream, s);
    else
        launch_hd<64>(a, G, grid, stream, s);
    if (a.nsplit > 1) hipLaunchKernelGGL(attn_fast_split_merge_kernel, dim3(a.m.Hq, a.B), dim3(a.m.hd), 0, s, a);
    return hipGetLastError();
}

int fast_attn_splits(int rows, int n_kv_heads, int max_pages_per_row, int n_cu, int cap) {
    const int blocks = rows * n_kv_heads;
    if (blocks <= 0 || blocks >= 2 * n_cu) return 1;  // enough blocks: one per (row, KV head)
    // short rows: a split saves less than the merge launch costs (one row of 512 positions, 8 KV
    // heads: 13.0 us in one block per KV head, 10.7 in two and 4.7 for the merge).  With 48 to 63 pages
    // of capacity rows that fill it would gain 1 to 3% of a two-layer step in splits at up to 16
    // rows, but rows at a quarter of it lose 2 to 3%, 32 rows lose 1 to 4% at any length and 17 rows of the
    // matrix-core verifier (whose split is that of 32) 5 to 7%
    if (max_pages_per_row < 64) return 1;
    int ns = (2 * n_cu + blocks - 1) / blocks;
    ns = ns < max_pages_per_row / 16 ? ns : max_pages_per_row / 16;
    // small batches: also shares of at most 64 pages, so that a long row does not leave
    // its one block working after the short rows' blocks are done
    const int by_length = (max_pages_per_row + 63) / 64;
    ns = ns > by_length ? ns : by_length;
    ns = ns < cap ? ns : cap;
    return ns < 1 ? 1 : ns;
}

}  // namespace mg
