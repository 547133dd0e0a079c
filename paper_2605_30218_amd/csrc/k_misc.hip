// k_misc.hip -- RMSNorm (with the item table and embedding gather of a forward's start), RoPE + K/V placement, SwiGLU, the
// top-1/top-2 margin gate, the K/V column repair, step bookkeeping, numerics probes.
#include "mg_device.h"
#include "mg_kernels.h"
#include "../../include/mg.h"

namespace mg {

// ------------------------------------------------------------------ RMSNorm
// ss = CDOT(x, x) (lane l owns groups l, l+64, ...; fma in element order; xor butterfly),
// m = ss / d, r = 1 / sqrt(m + eps), y_i = bf16((x_i * r) * gamma_i).
// The order of the sum leaves one wave per row for it, and a lone wave is bound by its own
// instruction stream (a vector instruction every 4 cycles: 8 per value for the output alone).  So
// four waves take a row: each forms the whole sum for itself (no exchange) and writes
// every fourth 64-group slice of the output, past a barrier, so that y may be x (a wave alone read
// the whole row before it wrote).  Against one wave per row: 4.9 and 6.6 us at 5 rows of
// 4096 values, 4.9 and 7.6 at 18 of 5120, 5.0 and 7.1 at 64 and 6.5 and 8.0 at 1000 of 4096.
constexpr int RMS_MAXG = 16;  // groups of 8 per lane: d <= 8192
constexpr int RMS_NW = 4;     // waves per row

// one row by this wave: src -> y (and xout, if not NULL, gets a copy of src), slices part, part + RMS_NW, ...
__device__ __forceinline__ void rmsnorm_row(const uint16_t* src, const uint16_t* gamma, int d, float eps, int lane,
                                            int part, uint16_t* xout, uint16_t* y) {
    const uint4* xr = reinterpret_cast<const uint4*>(src);
    const uint4* gr = reinterpret_cast<const uint4*>(gamma);
    const int G = d >> 3;
    // everything is requested together, so the wave waits for memory once (the wave's own slices
    // twice: a register array indexed by `part` would live in scratch memory)
    constexpr int NO = RMS_MAXG / RMS_NW;
    uint4 xv[RMS_MAXG], xo[NO], gv[NO];
#pragma unroll
    for (int k = 0; k < RMS_MAXG; ++k)
        if (64 * k < G) xv[k] = xr[min(lane + 64 * k, G - 1)];
#pragma unroll
    for (int k = 0; k < NO; ++k)
        if (64 * RMS_NW * k < G) {
            const int gi = min(lane + 64 * (RMS_NW * k + part), G - 1);
            xo[k] = xr[gi];
            gv[k] = gr[gi];
        }
    float a = 0.0f;
#pragma unroll
    for (int k = 0; k < RMS_MAXG; ++k) {
        if (64 * k < G && lane + 64 * k < G) {
            const uint4 v = xv[k];
            const float e[8] = {bf_lo(v.x), bf_hi(v.x), bf_lo(v.y), bf_hi(v.y),
                                bf_lo(v.z), bf_hi(v.z), bf_lo(v.w), bf_hi(v.w)};
#pragma unroll
            for (int i = 0; i < 8; ++i) a = __builtin_fmaf(e[i], e[i], a);
        }
    }
    const float ss = butterfly_sum(a);
    const float m = ieee_div(ss, (float)d);
    const float r = ieee_div(1.0f, ieee_sqrt(m + eps));
    __syncthreads();  // every wave's loads of the row are before every store
    uint4* yr = reinterpret_cast<uint4*>(y);
#pragma unroll
    for (int k = 0; k < NO; ++k) {
        const int gi = lane + 64 * (RMS_NW * k + part);
        if (64 * RMS_NW * k < G && gi < G) {
            const uint4 v = xo[k], w = gv[k];
            uint4 o;
            o.x = pack_bf2((bf_lo(v.x) * r) * bf_lo(w.x), (bf_hi(v.x) * r) * bf_hi(w.x));
            o.y = pack_bf2((bf_lo(v.y) * r) * bf_lo(w.y), (bf_hi(v.y) * r) * bf_hi(w.y));
            o.z = pack_bf2((bf_lo(v.z) * r) * bf_lo(w.z), (bf_hi(v.z) * r) * bf_hi(w.z));
            o.w = pack_bf2((bf_lo(v.w) * r) * bf_lo(w.w), (bf_hi(v.w) * r) * bf_hi(w.w));
            yr[gi] = o;
            if (xout) reinterpret_cast<uint4*>(xout)[gi] = v;
        }
    }
}

__global__ __launch_bounds__(64 * RMS_NW) void rmsnorm_kernel(const uint16_t* x, const uint16_t* __restrict__ g,
                                                              RowCount rc, int d, float eps, uint16_t* y) {
    const int row = blockIdx.x;
    if (row >= rc.get()) return;
    rmsnorm_row(x + (size_t)row * d, g, d, eps, threadIdx.x & 63, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nullptr,
                y + (size_t)row * d);
}

hipError_t launch_rmsnorm(const uint16_t* x, const uint16_t* gamma, int n_host, const int32_t* n_dev, int cap, int d,
                          float eps, uint16_t* y, hipStream_t s) {
    const int rows = n_dev ? cap : n_host;
    if (rows <= 0) return hipSuccess;
    if (d % 8 || d / 8 > 64 * RMS_MAXG) return hipErrorInvalidValue;
    RowCount rc{n_dev, n_host, cap};
    hipLaunchKernelGGL(rmsnorm_kernel, dim3(rows), dim3(64 * RMS_NW), 0, s, x, gamma, rc, d, eps, y);
    return hipGetLastError();
}

// The start of a canonical forward, one block per item: its entry of the item table (tab[i][0] =
// its position p, tab[i][1 + k] = its row's page of slot min(k, p / 16)), x[i] = embed[token of
// item i] and h[i] = RMSNorm(x[i]) (three launches of 4 to 6 us before).
__global__ __launch_bounds__(64 * RMS_NW) void first_norm_kernel(Items it, const uint16_t* __restrict__ E,
                                                         const uint16_t* __restrict__ g, int d, float eps, int mpr,
                                                         int32_t* __restrict__ tab, uint16_t* __restrict__ x,
                                                         uint16_t* __restrict__ h) {
    const int i = blockIdx.x;
    if (i >= items_n(it)) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = items_row(it, i), p = items_pos(it, i);
    const int32_t* ptab = it.page_table + (size_t)r * mpr;
    int32_t* tb = tab + (size_t)i * (1 + mpr);
    if (threadIdx.x == 0) tb[0] = p;
    for (int k = threadIdx.x; k < mpr; k += 64 * RMS_NW) tb[1 + k] = ptab[min(k, p >> 4)];
    rmsnorm_row(E + (size_t)items_tok(it, i) * d, g, d, eps, threadIdx.x & 63, wave, x + (size_t)i * d,
                   h + (size_t)i * d);
}

hipError_t launch_first_norm(const Items& it, const ModelDims& m, const uint16_t* embed, const uint16_t* gamma,
                             int32_t* itab, uint16_t* x, uint16_t* h, hipStream_t s) {
    if (it.n_host <= 0) return hipSuccess;
    if (m.d % 8 || m.d / 8 > 64 * RMS_MAXG) return hipErrorInvalidValue;
    hipLaunchKernelGGL(first_norm_kernel, dim3(it.n_host), dim3(64 * RMS_NW), 0, s, it, embed, gamma, m.d, m.eps,
                       m.max_pages_per_row, itab, x, h);
    return hipGetLastError();
}

// ------------------------------------------------------------------ RoPE + K/V placement
// Rotate-half RoPE: pair (i, i + hd/2) of every q and k head is rotated by the
// angle pos * theta^(-2i/hd), using the fp32 cos/sin table built on the host in
// float64.  q'_i = bf16(q_i c - q_(i+h) s), q'_(i+h) = bf16(q_(i+h) c + q_i s),
// products and sums separately rounded.  K' and V go to the verifier's own column
// (kv_col != NULL) or into the paged cache at the item's position.
__global__ __launch_bounds__(256) void rope_kv_kernel(Items it, ModelDims m, int layer, const uint16_t* __restrict__ qkv,
                                                      const float* __restrict__ cs, uint16_t* __restrict__ qrot,
                                                      uint16_t* __restrict__ kv_pool, uint16_t* __restrict__ kv_col) {
    const int i = blockIdx.x;
    if (i >= items_n(it)) return;
    const int r = items_row(it, i);
    const int pos = items_pos(it, i);
    const int hd = m.hd, h2 = hd / 2, Nq = m.Hq * hd, Nk = m.Hkv * hd;
    const uint16_t* src = qkv + (size_t)i * (Nq + 2 * Nk);
    const float* csp = cs + (size_t)pos * hd;  // [pos][i][cos, sin]
    uint16_t *kdst, *vdst;
    if (kv_col) {
        kdst = kv_col + ((size_t)i * m.L + layer) * 2 * Nk;
        vdst = kdst + Nk;
    } else {
        const int page = it.page_table[(size_t)r * m.max_pages_per_row + pos / m.page_size];
        const int slot = pos % m.page_size;
        // [layer][page][K|V][Hkv][page_size][hd]: head kh's row is at +kh*page_size*hd
        kdst = kv_pool + (((size_t)layer * m.n_pages + page) * 2) * (size_t)Nk * m.page_size + (size_t)slot * hd;
        vdst = kdst + (size_t)Nk * m.page_size;
    }
    const int kv_head_stride = kv_col ? hd : hd * m.page_size;
    // task = 8 consecutive pairs (i, i + hd/2) of one q or k head, or 8 values of v;
    // each thread's tasks are loaded together before any arithmetic
    const int gph = h2 / 8;                       // pair groups per head
    const int n_rot = (m.Hq + m.Hkv) * gph, n_v = Nk / 8;
    constexpr int TPT = 4;                        // tasks per thread per round
    for (int t0 = 0; t0 < n_rot + n_v; t0 += 256 * TPT) {
        uint4 lo[TPT], hi[TPT];
        float4 c4[TPT][4];
#pragma unroll
        for (int u = 0; u < TPT; ++u) {
            const int t = t0 + threadIdx.x + 256 * u;
            if (t < n_rot) {
                const int head = t / gph, ii = (t % gph) * 8;
                const uint16_t* sh = head < m.Hq ? src + head * hd : src + Nq + (head - m.Hq) * hd;
                lo[u] = *reinterpret_cast<const uint4*>(sh + ii);
                hi[u] = *reinterpret_cast<const uint4*>(sh + ii + h2);
#pragma unroll
                for (int q = 0; q < 4; ++q) c4[u][q] = *reinterpret_cast<const float4*>(csp + 2 * ii + 4 * q);
            } else if (t < n_rot + n_v) {
                lo[u] = *reinterpret_cast<const uint4*>(src + Nq + Nk + (t - n_rot) * 8);
            }
        }
#pragma unroll
        for (int u = 0; u < TPT; ++u) {
            const int t = t0 + threadIdx.x + 256 * u;
            if (t < n_rot) {
                const int head = t / gph, ii = (t % gph) * 8;
                const float a[8] = {bf_lo(lo[u].x), bf_hi(lo[u].x), bf_lo(lo[u].y), bf_hi(lo[u].y),
                                    bf_lo(lo[u].z), bf_hi(lo[u].z), bf_lo(lo[u].w), bf_hi(lo[u].w)};
                const float b[8] = {bf_lo(hi[u].x), bf_hi(hi[u].x), bf_lo(hi[u].y), bf_hi(hi[u].y),
                                    bf_lo(hi[u].z), bf_hi(hi[u].z), bf_lo(hi[u].w), bf_hi(hi[u].w)};
                const float cc[16] = {c4[u][0].x, c4[u][0].y, c4[u][0].z, c4[u][0].w, c4[u][1].x, c4[u][1].y,
                                      c4[u][1].z, c4[u][1].w, c4[u][2].x, c4[u][2].y, c4[u][2].z, c4[u][2].w,
                                      c4[u][3].x, c4[u][3].y, c4[u][3].z, c4[u][3].w};
                uint32_t o1[8], o2[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float c = cc[2 * e], sn = cc[2 * e + 1];
                    const float ac = a[e] * c, bs = b[e] * sn, bc = b[e] * c, as = a[e] * sn;
                    o1[e] = f2bf(ac - bs);
                    o2[e] = f2bf(bc + as);
                }
                const uint4 w1 = make_uint4(o1[0] | (o1[1] << 16), o1[2] | (o1[3] << 16), o1[4] | (o1[5] << 16),
                                            o1[6] | (o1[7] << 16));
                const uint4 w2 = make_uint4(o2[0] | (o2[1] << 16), o2[2] | (o2[3] << 16), o2[4] | (o2[5] << 16),
                                            o2[6] | (o2[7] << 16));
                uint16_t* dst = head < m.Hq ? qrot + (size_t)i * Nq + head * hd
                                            : kdst + (size_t)(head - m.Hq) * kv_head_stride;
                *reinterpret_cast<uint4*>(dst + ii) = w1;
                *reinterpret_cast<uint4*>(dst + ii + h2) = w2;
            } else if (t < n_rot + n_v) {
                const int e = (t - n_rot) * 8, head = e / hd, dd = e % hd;
                *reinterpret_cast<uint4*>(vdst + (size_t)head * kv_head_stride + dd) = lo[u];
            }
        }
    }
}

hipError_t launch_rope_kv(const Items& it, const ModelDims& m, int layer, const uint16_t* qkv, const float* rope_cs,
                          uint16_t* qrot, uint16_t* kv_pool, uint16_t* kv_col, hipStream_t s) {
    if (it.n_host <= 0) return hipSuccess;
    hipLaunchKernelGGL(rope_kv_kernel, dim3(it.n_host), dim3(256), 0, s, it, m, layer, qkv, rope_cs, qrot, kv_pool,
                       kv_col);
    return hipGetLastError();
}

// ------------------------------------------------------------------ top-1 / top-2
constexpr int TOP2_MAX_SLICES = 128;

// This thread's part of values j0 .. j1 - 1 of a row, merged over its wave (256 threads; 16-byte loads)
__device__ __forceinline__ Top2 top2_scan(const float* row, int V, int j0, int j1) {
    Top2 st{-__builtin_inff(), -__builtin_inff(), -1, 0};
    const int t = threadIdx.x;
    if ((V & 3) == 0) {  // slice is a multiple of 4, so are j0 and j1
        const float4* r4 = reinterpret_cast<const float4*>(row);
        for (int q = j0 / 4 + t; q < j1 / 4; q += 256) {
            const float4 v = r4[q];
            top2_push(st, v.x, 4 * q);
            top2_push(st, v.y, 4 * q + 1);
            top2_push(st, v.z, 4 * q + 2);
            top2_push(st, v.w, 4 * q + 3);
        }
    } else {
        for (int q = j0 + t; q < j1; q += 256) top2_push(st, row[q], q);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) st = top2_merge(st, top2_shfl(st, o));
    return st;
}

// row b's outputs from its merged state; whether its gate fires
__device__ __forceinline__ uint8_t top2_gate_row(const Top2& st, int b, const uint8_t* prot, float tau, int32_t* top1,
                                                 float* margin, uint8_t* gate) {
    const int i1 = st.i1 < 0 ? 0 : st.i1;
    const float g = st.nan ? __builtin_nanf("") : st.v1 - st.v2;
    int fire = 0;
    top1[b] = i1;
    if (margin) margin[b] = g;
    if (gate) {
        const int p = prot ? (prot[b] != 0) : 1;
        fire = p && !(g >= tau);
        gate[b] = (uint8_t)fire;
    }
    return (uint8_t)fire;
}

// the firing rows in increasing order and their count (thread t of a block of at least 256; rows
// 0..255 -> waves 0..3 of 64 rows: ballot, then prefix over the waves; one barrier)
__device__ __forceinline__ void top2_compact(int t, int nrows, const uint8_t* fire_s, int* wave_cnt, int32_t* gated_rows,
                                             int32_t* n_gated, int32_t* n_gated_host) {
    const int w = t >> 6, l = t & 63;
    const int f = (t < nrows) ? fire_s[t] : 0;  // t < 256 whenever t < nrows
    const unsigned long long bal = __ballot(f);
    if (w < 4 && l == 0) wave_cnt[w] = __popcll(bal);
    __syncthreads();
    if (w < 4) {
        int base = 0;
        for (int k = 0; k < w; ++k) base += wave_cnt[k];
        if (f) gated_rows[base + __popcll(bal & ((1ull << l) - 1ull))] = t;
        if (t == 0) {
            const int cnt = wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3];
            *n_gated = cnt;
            // mirror for a host that polls pinned memory (a system-scope release store; the
            // device-side consumers of the rows are ordered by the stream)
            if (n_gated_host) __hip_atomic_store(n_gated_host, cnt, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Stage 1: block (s, b) scans slice s of row b, merges its waves through LDS, and stores the
// slice's state.
__global__ __launch_bounds__(256) void top2_slice_kernel(int B, int V, int slice, const float* __restrict__ logits,
                                                         Top2* __restrict__ part, int nsl, const int32_t* n_dev) {
    const int s = blockIdx.x, b = blockIdx.y;
    const int nrows = n_dev ? min(max(*n_dev, 0), B) : B;
    if (b >= nrows) return;
    const int t = threadIdx.x;
    const Top2 st = top2_scan(logits + (size_t)b * V, V, s * slice, min((s + 1) * slice, V));
    __shared__ Top2 ws[4];
    if ((t & 63) == 0) ws[t >> 6] = st;
    __syncthreads();
    if (t == 0) part[(size_t)b * nsl + s] = top2_merge(top2_merge(ws[0], ws[1]), top2_merge(ws[2], ws[3]));
}

// Stage 2: one block of 1024 threads.  Row b's nsl slice states sit in nsl/2
// consecutive threads (2 states each, nsl a power of two, B * nsl <= 2048), merged
// by xor shuffles inside that lane group; then top1 / margin / gate, and the gated
// rows compacted in increasing order with per-wave ballots.
__global__ __launch_bounds__(1024) void top2_final_kernel(int B, const Top2* __restrict__ part, int nsl,
                                                          const uint8_t* __restrict__ prot, float tau, int32_t* top1,
                                                          float* margin, uint8_t* gate, int32_t* gated_rows,
                                                          int32_t* n_gated, int32_t* n_gated_host,
                                                          const int32_t* n_dev) {
    const int nrows = n_dev ? min(max(*n_dev, 0), B) : B;
    const int t = threadIdx.x;
    const int tpr = nsl / 2;            // threads per row (power of two, <= 64)
    const int b = t / tpr;
    const bool live = b < nrows;
    Top2 st{-__builtin_inff(), -__builtin_inff(), -1, 0};
    if (live) st = top2_merge(part[(size_t)b * nsl + 2 * (t % tpr)], part[(size_t)b * nsl + 2 * (t % tpr) + 1]);
    for (int o = 1; o < tpr; o <<= 1) st = top2_merge(st, top2_shfl(st, o));
    __shared__ uint8_t fire_s[256];
    __shared__ int wave_cnt[4];
    if (t % tpr == 0 && b < B) fire_s[b] = live ? top2_gate_row(st, b, prot, tau, top1, margin, gate) : 0;
    if (!gated_rows) return;
    __syncthreads();  // fire_s complete
    top2_compact(t, nrows, fire_s, wave_cnt, gated_rows, n_gated, n_gated_host);
}

// A slice state for another block of the same launch: agent-scope words, which go past the L2s of
// the XCDs by themselves
__device__ __forceinline__ void top2_store_agent(Top2* p, const Top2& st) {
    const unsigned w[4] = {__float_as_uint(st.v1), __float_as_uint(st.v2), (unsigned)st.i1, (unsigned)st.nan};
    unsigned* d = reinterpret_cast<unsigned*>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) __hip_atomic_store(d + k, w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ Top2 top2_load_agent(Top2* p) {
    unsigned w[4];
    unsigned* d = reinterpret_cast<unsigned*>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = __hip_atomic_load(d + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return Top2{__uint_as_float(w[0]), __uint_as_float(w[1]), (int)w[2], (int)w[3]};
}

// Both stages in one launch for up to 256 slice states (few rows, or a small vocabulary): the block
// that finishes last merges them (launch_top2 says when it is taken).  A state is stored past the L2 and waited for before the
// counter is incremented, and read after; a release fence instead writes back an XCD's L2 in every block
// (64 rows of 4096: 11.7 us of kernel time).  atomicInc wraps to 0 at the launch's own block count and every
// block count has a counter of its own, so a launch leaves its counter as it found it.
__global__ __launch_bounds__(256) void top2_single_kernel(int B, int V, int slice, const float* __restrict__ logits,
                                                          Top2* part, int nsl, unsigned* counters,
                                                          const uint8_t* __restrict__ prot, float tau, int32_t* top1,
                                                          float* margin, uint8_t* gate, int32_t* gated_rows,
                                                          int32_t* n_gated, int32_t* n_gated_host,
                                                          const int32_t* n_dev) {
    const int s = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
    const int nrows = n_dev ? min(max(*n_dev, 0), B) : B;
    __shared__ Top2 ws[4];
    __shared__ int last;
    if (b < nrows) {
        const Top2 st = top2_scan(logits + (size_t)b * V, V, s * slice, min((s + 1) * slice, V));
        if ((t & 63) == 0) ws[t >> 6] = st;
    }
    __syncthreads();
    if (t == 0) {
        if (b < nrows) top2_store_agent(&part[b * nsl + s], top2_merge(top2_merge(ws[0], ws[1]), top2_merge(ws[2], ws[3])));
        const unsigned total = gridDim.x * gridDim.y;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the state is stored
        last = atomicInc(counters + total, total - 1) == total - 1;
        asm volatile("" ::: "memory");
    }
    __syncthreads();
    if (!last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the states' loads stay behind the counter
    // state t of row t / nsl (nsl a power of two up to 64, B * nsl <= 256)
    const int row = t / nsl;
    Top2 st{-__builtin_inff(), -__builtin_inff(), -1, 0};
    if (row < nrows) st = top2_load_agent(&part[t]);
    for (int o = 1; o < nsl; o <<= 1) st = top2_merge(st, top2_shfl(st, o));
    __shared__ uint8_t fire_s[256];
    __shared__ int wave_cnt[4];
    fire_s[t] = 0;
    __syncthreads();
    if (t % nsl == 0 && row < nrows) fire_s[row] = top2_gate_row(st, row, prot, tau, top1, margin, gate);
    if (!gated_rows) return;
    __syncthreads();
    top2_compact(t, nrows, fire_s, wave_cnt, gated_rows, n_gated, n_gated_host);
}

int top2_slices(int B, int V) {
    int nsl = 2;
    while (nsl * 2 <= TOP2_MAX_SLICES && (nsl * 2) * (B > 0 ? B : 1) <= 2048 && (V + nsl * 2 - 1) / (nsl * 2) >= 1024)
        nsl *= 2;
    return nsl;
}

// slices of a single-launch gate, or 0: at most 64 (one row's states in one wave) and 256 states, no
// slice more than 4 times as long as the two-launch form's (18 rows of 32000 in 8 instead of 32: 8.2 us
// against 10.1) or above 4096 values (8 rows of 152064 in slices of 4752: 10.3 against 10.1).  Rows that
// are not 16-byte multiples are read by the word, which takes about 5.4 us + 13.7 ns a state + 0.66 ns a
// value of a slice (8 rows of 128257, 256 states of 4012: 11.6; 6 rows 10.7; 16 of 50257, 256 of 3144: 10.9;
// 4 of 128257, 256 of 2008: 10.3), against 10.3 to 10.9 for the calls of two launches
static int top2_single_slices(int B, int V) {
    const int two = top2_slices(B, V);
    int nsl = two < 64 ? two : 64;
    while (nsl > 1 && nsl * B > 256) nsl /= 2;
    if (V % 4 && 21L * nsl * B + V / nsl > 7700) return 0;
    return nsl * B <= 256 && nsl * 4 >= two && V <= 4096L * nsl ? nsl : 0;
}

size_t top2_ws_bytes(int B, int V) {
    return B <= 0 ? 0 : (size_t)top2_slices(B, V) * B * sizeof(Top2);
}

static bool stream_captures(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st == hipStreamCaptureStatusActive;
}

// The arrivals at the one counter come one after the other, about 9 ns each.  Up to 64 states the
// single launch takes no more of the GPU than the two (in a graph, back to back: one row of 128256
// values 7.5 against 7.7 us, 16 rows of 4096 6.4 against 6.6, 4 of 32000 7.1 against 7.3); above, it takes more (32 rows of
// 4096 7.1 against 6.6, 64 of them 8.7 against 6.8, 8 of 128256 10.4 against 8.1) and pays only where the
// host's launches set the time, which is a gate called by itself outside a graph (a call: 8.1 against 10.2
// us, 8.5 against 10.3, 10.1 against 10.3), not the last step of a verifier call (alone = false).  The same
// for slices above 2048 values read by the word (one row of 152063 8.1 against 7.2 in a graph).
hipError_t launch_top2(int B, int V, const float* logits, const uint8_t* prot, float tau, int32_t* top1, float* margin,
                       uint8_t* gate, int32_t* gated_rows, int32_t* n_gated, int32_t* n_gated_host, void* part_ws,
                       unsigned* counters, const int32_t* n_dev, bool alone, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    if (B > 256) return hipErrorInvalidValue;
    Top2* part = static_cast<Top2*>(part_ws);
    const int one = top2_single_slices(B, V);
    const bool even = one * B <= 64 && !(V % 4 && V > 2048L * one);
    if (one && (even || (alone && !stream_captures(s)))) {
        const int slice = ((V + one - 1) / one + 3) & ~3;
        hipLaunchKernelGGL(top2_single_kernel, dim3(one, B), dim3(256), 0, s, B, V, slice, logits, part, one, counters,
                           prot, tau, top1, margin, gate, gated_rows, n_gated, n_gated_host, n_dev);
        return hipGetLastError();
    }
    const int nsl = top2_slices(B, V);
    int slice = (V + nsl - 1) / nsl;
    slice = (slice + 3) & ~3;
    hipLaunchKernelGGL(top2_slice_kernel, dim3(nsl, B), dim3(256), 0, s, B, V, slice, logits, part, nsl, n_dev);
    hipLaunchKernelGGL(top2_final_kernel, dim3(1), dim3(1024), 0, s, B, part, nsl, prot, tau, top1, margin, gate,
                       gated_rows, n_gated, n_gated_host, n_dev);
    return hipGetLastError();
}

// ------------------------------------------------------------------ single-column repair
// One block per listed row.  The decision is taken once (v_tok vs top1, read
// before anything is written, so emitted may alias top1); on a mismatch the
// verifier column [L][K|V][Hkv][hd] is copied to the row's current position in
// every layer, then emitted and the repair counter are updated.
__global__ void gather_rows_kernel(int n, const int32_t* __restrict__ rows, const int32_t* __restrict__ tokens,
                                   const int32_t* __restrict__ positions, const int32_t* __restrict__ page_table,
                                   int maxp, int32_t* __restrict__ out_tok, int32_t* __restrict__ out_pos,
                                   int32_t* __restrict__ out_pt) {
    const int i = blockIdx.x;
    if (i >= n) return;
    const int r = rows[i];
    if (threadIdx.x == 0) {
        out_tok[i] = tokens[r];
        out_pos[i] = positions[r];
    }
    for (int k = threadIdx.x; k < maxp; k += blockDim.x) out_pt[(size_t)i * maxp + k] = page_table[(size_t)r * maxp + k];
}

hipError_t launch_gather_rows(int n, const int32_t* rows, const int32_t* tokens, const int32_t* positions,
                              const int32_t* page_table, int maxp, int32_t* out_tok, int32_t* out_pos, int32_t* out_pt,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_rows_kernel, dim3(n), dim3(256), 0, s, n, rows, tokens, positions, page_table, maxp,
                       out_tok, out_pos, out_pt);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void repair_kernel(RowCount rc, const int32_t* __restrict__ rows,
                                                     const int32_t* __restrict__ positions,
                                                     const int32_t* __restrict__ page_table, const int32_t* top1,
                                                     const int32_t* __restrict__ v_tok,
                                                     const uint16_t* __restrict__ v_kvcol, ModelDims m,
                                                     uint16_t* __restrict__ kv_pool, int32_t* emitted,
                                                     int32_t* n_repaired, int action) {
    const int i = blockIdx.x;
    if (i >= rc.get()) return;
    __shared__ int decide[2];
    const int r = rows[i];
    if (threadIdx.x == 0) {
        decide[0] = v_tok[i];
        // the method copies on a disagreement; the variants never copy (token only) or
        // always copy
        decide[1] = action == MG_REPAIR_COPY_ALWAYS ? 1 : action == MG_REPAIR_TOKEN_ONLY ? 0 : (v_tok[i] != top1[r]);
    }
    __syncthreads();
    const int vt = decide[0];
    if (decide[1]) {
        const int pos = positions[r];
        const int page = page_table[(size_t)r * m.max_pages_per_row + pos / m.page_size];
        const int slot = pos % m.page_size;
        const int hd = m.hd, per_head = hd / 8;  // uint4 per head row
        const int segs = m.L * 2 * m.Hkv;
        const uint4* src = reinterpret_cast<const uint4*>(v_kvcol + (size_t)i * segs * hd);
        for (int t = threadIdx.x; t < segs * per_head; t += blockDim.x) {
            const int seg = t / per_head, u = t % per_head;
            const int layer = seg / (2 * m.Hkv), kv = (seg / m.Hkv) % 2, kh = seg % m.Hkv;
            uint16_t* dst = kv_pool + ((((size_t)layer * m.n_pages + page) * 2 + kv) * m.Hkv + kh) * (size_t)m.page_size * hd +
                            (size_t)slot * hd;
            reinterpret_cast<uint4*>(dst)[u] = src[t];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        emitted[r] = vt;
        if (decide[1]) atomicAdd(n_repaired, 1);
    }
}

hipError_t launch_repair(int n_host, const int32_t* n_dev, int cap, const int32_t* rows, const int32_t* positions,
                         const int32_t* page_table, const int32_t* top1, const int32_t* v_tok, const uint16_t* v_kvcol,
                         const ModelDims& m, uint16_t* kv_pool, int32_t* emitted, int32_t* n_repaired, int action, hipStream_t s) {
    const int grid = n_dev ? cap : n_host;
    if (grid <= 0) return hipSuccess;
    RowCount rc{n_dev, n_host, cap};
    hipLaunchKernelGGL(repair_kernel, dim3(grid), dim3(256), 0, s, rc, rows, positions, page_table, top1, v_tok,
                       v_kvcol, m, kv_pool, emitted, n_repaired, action);
    return hipGetLastError();
}

// ------------------------------------------------------------------ bookkeeping
__global__ void advance_kernel(int B, const int32_t* __restrict__ emitted, int32_t* tokens, int32_t* positions) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) {
        tokens[b] = emitted[b];
        positions[b] += 1;
    }
}

hipError_t launch_advance(int B, const int32_t* emitted, int32_t* tokens, int32_t* positions, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(advance_kernel, dim3((B + 255) / 256), dim3(256), 0, s, B, emitted, tokens, positions);
    return hipGetLastError();
}

// ------------------------------------------------------------------ numerics probes
__global__ void probe_bf16_kernel(int64_t n, const float* in, uint16_t* out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (uint16_t)f2bf(in[i]);
}
__global__ void probe_exp_kernel(int64_t n, const float* in, float* out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = canon_exp(in[i]);
}
__global__ void probe_divsqrt_kernel(int64_t n, const float* a, const float* b, float* q, float* r) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        q[i] = ieee_div(a[i], b[i]);
        r[i] = ieee_sqrt(a[i]);
    }
}

// plain 16-byte copy: reads and writes n16 * 16 bytes once (counter calibration)
__global__ __launch_bounds__(256) void copy16_kernel(int64_t n16, const uint4* __restrict__ src, uint4* __restrict__ dst) {
    // four independent 16-byte loads in flight per thread before the stores
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const uint4 a = src[i], b = src[i + stride], c = src[i + 2 * stride], d = src[i + 3 * stride];
        dst[i] = a;
        dst[i + stride] = b;
        dst[i + 2 * stride] = c;
        dst[i + 3 * stride] = d;
    }
    for (; i < n16; i += stride) dst[i] = src[i];
}

hipError_t launch_copy16(int64_t n16, const void* src, void* dst, hipStream_t s) {
    if (n16 <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy16_kernel, dim3(2048), dim3(256), 0, s, n16, static_cast<const uint4*>(src),
                       static_cast<uint4*>(dst));
    return hipGetLastError();
}

// Streaming read of n16 16-byte words (eight loads in flight per thread, grid-stride): the
// reference for the HBM read rate the weight- and K/V-streaming kernels could reach.  Each
// block stores the xor of its words to sink[block], which keeps every load.
constexpr int READ_STREAM_BLOCKS = 16384;
__global__ __launch_bounds__(256) void read_stream_kernel(int64_t n16, const uint4* __restrict__ src,
                                                          uint32_t* __restrict__ sink) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    uint32_t acc = 0;
    for (; i + 7 * stride < n16; i += 8 * stride) {
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[i + u * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (; i < n16; i += stride) {
        const uint4 v = src[i];
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    __shared__ uint32_t red[4];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc ^= __shfl_xor(acc, o, MG_WAVE);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) sink[blockIdx.x] = red[0] ^ red[1] ^ red[2] ^ red[3];
}

int read_stream_blocks() { return READ_STREAM_BLOCKS; }

hipError_t launch_read_stream(int64_t n16, const void* src, uint32_t* sink, hipStream_t s) {
    if (n16 <= 0) return hipSuccess;
    hipLaunchKernelGGL(read_stream_kernel, dim3(READ_STREAM_BLOCKS), dim3(256), 0, s, n16,
                       static_cast<const uint4*>(src), sink);
    return hipGetLastError();
}

static int probe_grid(int64_t n) { return (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096); }

hipError_t launch_probe_bf16(int64_t n, const float* in, uint16_t* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(probe_bf16_kernel, dim3(probe_grid(n)), dim3(256), 0, s, n, in, out);
    return hipGetLastError();
}
hipError_t launch_probe_exp(int64_t n, const float* in, float* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(probe_exp_kernel, dim3(probe_grid(n)), dim3(256), 0, s, n, in, out);
    return hipGetLastError();
}
hipError_t launch_probe_divsqrt(int64_t n, const float* a, const float* b, float* q, float* r, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(probe_divsqrt_kernel, dim3(probe_grid(n)), dim3(256), 0, s, n, a, b, q, r);
    return hipGetLastError();
}

typedef float probe_v16f __attribute__((ext_vector_type(16)));

// The instruction the matrix-core canonical GEMV (k_gemv_mfma.hip) relies on, bare: per instance t (one wave),
// D = v_mfma_f32_16x16x1_4b_f32(a[t][lane], b[t][lane], C) with C and D [t][register][lane]
__global__ __launch_bounds__(64) void probe_mfma_fma_kernel(const float* __restrict__ a, const float* __restrict__ b,
                                                            const float* __restrict__ c, float* __restrict__ d) {
    const size_t t = blockIdx.x;
    const int lane = threadIdx.x;
    probe_v16f acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = c[(t * 16 + r) * 64 + lane];
    acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a[t * 64 + lane], b[t * 64 + lane], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) d[(t * 16 + r) * 64 + lane] = acc[r];
}

hipError_t launch_probe_mfma_fma(int n_inst, const float* a, const float* b, const float* c, float* d, hipStream_t s) {
    if (n_inst <= 0) return hipSuccess;
    hipLaunchKernelGGL(probe_mfma_fma_kernel, dim3(n_inst), dim3(64), 0, s, a, b, c, d);
    return hipGetLastError();
}

// one v_mfma_f32_4x4x1_16b_f32 per wave: a, b [n][64], c, d [n][4][64]
typedef float probe_v4f __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(64) void probe_mfma4_fma_kernel(const float* __restrict__ a, const float* __restrict__ b,
                                                             const float* __restrict__ c, float* __restrict__ d) {
    const size_t t = blockIdx.x;
    const int lane = threadIdx.x;
    probe_v4f acc;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = c[(t * 4 + r) * 64 + lane];
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a[t * 64 + lane], b[t * 64 + lane], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) d[(t * 4 + r) * 64 + lane] = acc[r];
}

hipError_t launch_probe_mfma4_fma(int n_inst, const float* a, const float* b, const float* c, float* d, hipStream_t s) {
    if (n_inst <= 0) return hipSuccess;
    hipLaunchKernelGGL(probe_mfma4_fma_kernel, dim3(n_inst), dim3(64), 0, s, a, b, c, d);
    return hipGetLastError();
}

}  // namespace mg
