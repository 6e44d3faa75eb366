// HIP kernels of the Polya-urn partially collapsed LDA sampler for gfx950.
//
// Algorithm 2 of the paper (Section 3): every sweep draws each topic row
// phi_k ~ PPU(n_k + beta) (the Phi-step), then every token's topic from
// P(z_i = k) propto phi_{k,v(i)} (alpha_k + m^{-i}_{d,k}) (the z-step), and the
// counts n, m are rebuilt from z.  Section 3.4 gives the Poisson draws (alias
// tables for rates beta + l, l <= L; rounded Gaussian above), Section 3.5 the
// a/b split of the token conditional and the doubly sparse b-sum.
//
// Layouts in HBM (all word-major, so one word's column is contiguous):
//   n[v*K + k]                                  dense counts
//   gam                                          the draws, each word's row in
//     the narrowest format that holds it; phid[v*K + k] fp32 values instead
//     where Phi has no draws
//   colptr[v] .. colptr[v+1]                    CSC of Phi's nonzeros by word,
//     ctopic (u16, ascending), cphi (f32), calias (u64: thr | topic << 32 |
//     alias topic << 48)
//   doc_off[d] .. doc_off[d+1]                  CSR tokens, words (i32), z (u16)
#include <hip/hip_runtime.h>

#include "device.h"
#include "internal.h"

namespace pulda {

// ---------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------
__global__ void fill_u32_kernel(uint32_t *p, uint32_t value, int64_t count)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

__global__ void fill_u64_kernel(unsigned long long *p, unsigned long long value, int64_t count)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

static int grid_for(int64_t n, int block, int cap = 65536)
{
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t value, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    fill_u32_kernel<<<grid_for(count, 256, 16384), 256, 0, s>>>(p, value, count);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, unsigned long long value, int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    fill_u64_kernel<<<grid_for(count, 256, 16384), 256, 0, s>>>(p, value, count);
    return hipGetLastError();
}

// LDS accesses of the wave before and after are kept in this order (LDS
// executes a wave's instructions in order; only the compiler is held)
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// byte offset of word v's row of draws from gam
__device__ __forceinline__ uint32_t draws_offset(const DevModel &m, uint32_t fmt, int32_t v)
{
    return fmt == ROW_8 ? m.row_base[0] + (uint32_t)v * m.row_step[0]
                        : (fmt == ROW_16 ? m.row_base[1] + (uint32_t)v * m.row_step[1] : (uint32_t)v * m.row_step[2]);
}

// draw of topic k in word v's row of format fmt (Phi of draws)
__device__ __forceinline__ uint32_t row_draw(const DevModel &m, uint32_t fmt, int32_t v, int32_t k)
{
    const uint8_t *row = m.gam + draws_offset(m, fmt, v);
    if (fmt == ROW_8) return row[k];
    if (fmt == ROW_16) return ((const uint16_t *)row)[k];
    return ((const uint32_t *)row)[k];
}

// phi_kv = fp32(gamma / S_k), the quotient in fp64; or the loaded value
__device__ __forceinline__ float phi_at(const DevModel &m, int32_t v, int32_t k)
{
    if (m.values) return m.phid[(int64_t)v * m.K + k];
    const uint32_t x = row_draw(m, m.wrec[v].y >> 30, v, k);
    return x ? (float)((double)x / (double)m.S[k]) : 0.0f;
}

// ---------------------------------------------------------------------------
// exclusive scans (three passes: block sums, scan of block sums, add-back)
// ---------------------------------------------------------------------------
constexpr int SCAN_BLOCK = 1024;

template <typename Tin>
__global__ void scan_block_sums(const Tin *in, int64_t n, long long *bsum)
{
    __shared__ long long part[SCAN_BLOCK / 64];
    int64_t i = blockIdx.x * (int64_t)SCAN_BLOCK + threadIdx.x;
    long long x = i < n ? (long long)in[i] : 0;
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long t = 0;
        for (int w = 0; w < SCAN_BLOCK / 64; ++w) t += part[w];
        bsum[blockIdx.x] = t;
    }
}

__global__ void scan_sums_serial(long long *bsum, int64_t nb, long long *total)
{
    // one block: each thread scans a contiguous chunk, then chunk offsets are combined
    __shared__ long long chunk[1024];
    int64_t per = (nb + blockDim.x - 1) / blockDim.x;
    int64_t a = threadIdx.x * per, b = a + per < nb ? a + per : nb;
    long long t = 0;
    for (int64_t i = a; i < b; ++i) t += bsum[i];
    chunk[threadIdx.x] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long run = 0;
        for (int j = 0; j < (int)blockDim.x; ++j) {
            long long c = chunk[j];
            chunk[j] = run;
            run += c;
        }
        if (total) *total = run;
    }
    __syncthreads();
    long long run = chunk[threadIdx.x];
    for (int64_t i = a; i < b; ++i) {
        long long c = bsum[i];
        bsum[i] = run;
        run += c;
    }
}

template <typename Tin, typename Tout>
__global__ void scan_apply(const Tin *in, int64_t n, const long long *boff, Tout *out)
{
    __shared__ long long wsum[SCAN_BLOCK / 64];
    int64_t i = blockIdx.x * (int64_t)SCAN_BLOCK + threadIdx.x;
    long long x = i < n ? (long long)in[i] : 0;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    long long incl = x;
    for (int o = 1; o < 64; o <<= 1) {
        long long y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    long long before = boff[blockIdx.x];
    for (int j = 0; j < w; ++j) before += wsum[j];
    if (i < n) out[i] = (Tout)(before + incl - x);
    if (i == n - 1) out[n] = (Tout)(before + incl);
}

template <typename Tin, typename Tout>
static hipError_t scan_excl(const Tin *in, Tout *out, int64_t n, long long *scratch, long long *total,
                            hipStream_t s)
{
    // out has n + 1 entries; scratch holds ceil(n / SCAN_BLOCK) entries
    if (n <= 0) {
        scan_sums_serial<<<1, 64, 0, s>>>(scratch, 0, total);
        return hipGetLastError();
    }
    int64_t nb = (n + SCAN_BLOCK - 1) / SCAN_BLOCK;
    scan_block_sums<Tin><<<(unsigned)nb, SCAN_BLOCK, 0, s>>>(in, n, scratch);
    scan_sums_serial<<<1, 1024, 0, s>>>(scratch, nb, total);
    scan_apply<Tin, Tout><<<(unsigned)nb, SCAN_BLOCK, 0, s>>>(in, n, scratch, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// corpus validation: monotone offsets from 0 to N, word ids in [0, V),
// document lengths within the 16-bit per-document count range
// ---------------------------------------------------------------------------
__global__ void validate_kernel(const int64_t *doc_off, int64_t D, const int32_t *words, int64_t N, int32_t V,
                                int32_t *err)
{
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; d < D; d += stride) {
        int64_t a = doc_off[d], b = doc_off[d + 1];
        if (b < a || a < 0 || b > N) atomicAdd(&err[0], 1);
        else if (b - a > 65535) atomicAdd(&err[2], 1);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (doc_off[0] != 0 || doc_off[D] != N) atomicAdd(&err[0], 1);
    }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += stride) {
        int32_t w = words[i];
        if (w < 0 || w >= V) atomicAdd(&err[1], 1);
    }
}

hipError_t launch_validate(const DevCorpus &c, int32_t V, int32_t *err, hipStream_t s)
{
    validate_kernel<<<grid_for(c.N > c.D ? c.N : c.D, 256, 8192), 256, 0, s>>>(c.doc_off, c.D, c.words, c.N, V, err);
    return hipGetLastError();
}

// caller-supplied state and Phi: every topic below K, columns well formed
__global__ void check_u16_below_kernel(const uint16_t *x, int64_t n, uint32_t limit, int32_t *err)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        if (x[i] >= limit) atomicAdd(err, 1);
}

hipError_t launch_check_u16_below(const uint16_t *x, int64_t n, uint32_t limit, int32_t *err, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    check_u16_below_kernel<<<grid_for(n, 256, 8192), 256, 0, s>>>(x, n, limit, err);
    return hipGetLastError();
}

__global__ void check_phi_kernel(const int64_t *colptr, int32_t V, const uint16_t *topic, const uint16_t *alias_topic,
                                 uint32_t K, int32_t *err)
{
    const int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= V) return;
    const int lane = __lane_id();
    const int64_t a = colptr[v], b = colptr[v + 1];
    if (b < a || b - a > (int64_t)K) {
        if (lane == 0) atomicAdd(err, 1);
        return;
    }
    for (int64_t e = a + lane; e < b; e += 64) {
        const bool ok = topic[e] < K && alias_topic[e] < K && (e == a || topic[e - 1] < topic[e]);
        if (!ok) atomicAdd(err, 1);
    }
}

hipError_t launch_check_phi(const int64_t *colptr, int32_t V, const uint16_t *topic, const uint16_t *alias_topic,
                            uint32_t K, int32_t *err, hipStream_t s)
{
    check_phi_kernel<<<(V + 3) / 4, 256, 0, s>>>(colptr, V, topic, alias_topic, K, err);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// initial state: z_i uniform on {0..K-1}
// ---------------------------------------------------------------------------
__global__ void init_z_kernel(uint16_t *z, int64_t N, int32_t K, uint32_t key0, uint32_t key1)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x) {
        r4 r = philox((uint32_t)i, (uint32_t)((uint64_t)i >> 32), 0u, TAG_INIT, key0, key1);
        z[i] = (uint16_t)scale32(r.x, (uint32_t)K);
    }
}

hipError_t launch_init_z(const DevCorpus &c, int32_t K, uint32_t key0, uint32_t key1, hipStream_t s)
{
    if (c.N == 0) return hipSuccess;
    init_z_kernel<<<grid_for(c.N, 256, 16384), 256, 0, s>>>(c.z, c.N, K, key0, key1);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// count rebuild from z (Table 1): n[v*K + k] += 1 for every token
// ---------------------------------------------------------------------------
__global__ void count_tokens_kernel(const int32_t *words, const uint16_t *z, int64_t N, int32_t K, int32_t *n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&n[(int64_t)words[i] * K + z[i]], 1);
}

hipError_t launch_count_rebuild(const DevCorpus &c, const DevModel &m, hipStream_t s)
{
    hipError_t e = launch_fill_u32((uint32_t *)m.n, 0u, (int64_t)m.V * m.K, s);
    if (e != hipSuccess) return e;
    if (c.N == 0) return hipSuccess;
    count_tokens_kernel<<<grid_for(c.N, 256, 16384), 256, 0, s>>>(c.words, c.z, c.N, m.K, m.n);
    return hipGetLastError();
}

// column sums of a word-major V x K table: out[k] += sum_v dense[v*K + k]

__global__ void row_sums_kernel(const int32_t *dense, int32_t V, int32_t K, unsigned long long *out)
{
    const int32_t v0 = blockIdx.x * ROWSUM_COLS;
    const int32_t v1 = v0 + ROWSUM_COLS < V ? v0 + ROWSUM_COLS : V;
    for (int32_t k = threadIdx.x; k < K; k += blockDim.x) {
        unsigned long long t = 0;
        int32_t v = v0;
        // eight rows' loads in flight before they are added
        for (; v + 8 <= v1; v += 8) {
            uint32_t x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = (uint32_t)dense[(int64_t)(v + j) * K + k];
#pragma unroll
            for (int j = 0; j < 8; ++j) t += x[j];
        }
        for (; v < v1; ++v) t += (unsigned long long)(uint32_t)dense[(int64_t)v * K + k];
        if (t) atomicAdd(&out[k], t);
    }
}

hipError_t launch_row_sums(const int32_t *dense, int32_t V, int32_t K, unsigned long long *out, hipStream_t s)
{
    hipError_t e = launch_fill_u64(out, 0ull, K, s);
    if (e != hipSuccess) return e;
    row_sums_kernel<<<(V + ROWSUM_COLS - 1) / ROWSUM_COLS, 256, 0, s>>>(dense, V, K, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Phi-step, part 1 (Section 3.4): one wave per word column v.
//   counted cells (n_kv = l >= 1) draw Pois(beta + l): alias table of l for
//   l <= L, rounded Gaussian for l > L;
//   zero-count cells draw Pois(beta); the nonzero ones are reached by
//   geometric jumps (gap = floor(-ln(1-U)/beta)), 64 jumps per round, their
//   positions by a wave prefix sum of the jump lengths.
// Most words count few topics, so the counted cells are first listed: the
// random numbers and table reads then run on full waves, not on the few
// lanes of each 64 cells (the cells past the tables are listed once more).
// The draws of a word leave as its narrowest row (8, 16 or 32 bits a topic),
// the only dense table written; a block adds its words' draws by topic in
// LDS and writes one row of partial sums for phi_sums_kernel.
// Measured at V = 141,000, K = 1000 and 738M tokens (the counts are 564 MB):
// 400 us, from 650 us for cells drawn where they lie and 32-bit rows, plus
// 140 us for a pass over the draws that added them up.  It is bound by VALU
// issue (905 instructions a word, half the time: the Philox rounds) and, at
// 20 waves a CU for the LDS of K topics, by waits for a word's tables; loading
// the next word's counts ahead gave nothing.
// ---------------------------------------------------------------------------
// bytes of LDS per topic: the block's sums, and a wave's draws and list
constexpr int32_t PHI_SUM_BYTES = 8, PHI_WAVE_BYTES = 6;
constexpr int PHI_DRAW_WAVES = 4;   // per block

__global__ void __launch_bounds__(64 * PHI_DRAW_WAVES) phi_draw_kernel(DevModel m, unsigned long long *part,
                                                                       unsigned long long *stats)
{
    constexpr int WAVES = PHI_DRAW_WAVES;
    extern __shared__ __align__(16) uint8_t phi_lds[];
    const uint32_t t = *m.tptr;
    const int lane = __lane_id();
    const int w = threadIdx.x >> 6;
    const int32_t K = m.K, kpad = m.ks16;
    unsigned long long *sum = (unsigned long long *)phi_lds;
    int32_t *g = (int32_t *)(phi_lds + PHI_SUM_BYTES * (size_t)kpad) + w * kpad;
    uint16_t *lst = (uint16_t *)(phi_lds + (PHI_SUM_BYTES + 4 * WAVES) * (size_t)kpad) + w * kpad;
    if (blockIdx.x == 0 && threadIdx.x == 0 && stats) stats[ST_EMPTY_ROWS] = 0;
    for (int32_t k = threadIdx.x; k < K; k += 64 * WAVES) sum[k] = 0;
    __syncthreads();
    const double two_pi = 6.283185307179586476925286766559;
    const bool vec = m.beta_v != nullptr;
    const double tb = vec ? 0.0 : m.beta;
    const uint64_t below = (1ull << lane) - 1ull;
    auto put = [&](int32_t k, int32_t x) {
        g[k] = x;
        if (x > 0) atomicAdd(&sum[k], (unsigned long long)x);
    };
    for (int32_t v = blockIdx.x * WAVES + w; v < m.V; v += gridDim.x * WAVES) {
        const int32_t *ncol = m.n + (int64_t)v * K;
        // per-word priors: the tables are of integer rates l and every cell's
        // Pois(beta_v) part comes from the prior marks below, added to its draw
        const double bv = vec ? m.beta_v[v] : m.beta;
        const uint32_t *T = m.ztp_tab + (vec ? m.ztp_off[v] : 0);
        const int32_t nT = vec ? m.ztp_off[v + 1] - m.ztp_off[v] : m.ztp_n;

        // the counts, PR rounds of 64 cells in flight; -1 marks a zero-count cell
        constexpr int PR = 16;
        int32_t n = 0;
        for (int32_t kb = 0; kb < kpad; kb += 64 * PR) {
            int32_t lv[PR];
#pragma unroll
            for (int u = 0; u < PR; ++u) {
                const int32_t k = kb + 64 * u + lane;
                lv[u] = k < K ? ncol[k] : 0;
            }
#pragma unroll
            for (int u = 0; u < PR; ++u) {
                if (kb + 64 * u >= kpad) break;
                const int32_t k = kb + 64 * u + lane;
                g[k] = lv[u] > 0 ? lv[u] : -1;
                const uint64_t bal = __builtin_amdgcn_ballot_w64(lv[u] > 0);
                if (lv[u] > 0) lst[n + __builtin_popcountll(bal & below)] = (uint16_t)k;
                n += __builtin_popcountll(bal);
            }
        }
        lds_order();
        // rates with a table, U rounds of 64 cells at a time: their tables'
        // offsets, then their entries are loaded for all rounds before any is
        // used.  Slot j of the alias table of rate l, kept when r.y is below
        // its threshold, else its alias
        constexpr int U = 4;
        int32_t far = 0;   // cells past the tables, listed from the front again
        for (int32_t i0 = 0; i0 < n; i0 += 64 * U) {
            int32_t kk[U], lo[U], hi[U];
            bool tab[U], past[U];
            uint32_t jv[U], ry[U];
            uint64_t ev[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t i = i0 + 64 * u + lane;
                kk[u] = i < n ? lst[i] : 0;
                const int32_t l = i < n ? g[kk[u]] : 0;
                tab[u] = l > 0 && l <= m.L;
                past[u] = l > m.L;
                lo[u] = tab[u] ? m.pois_off[l] : 0;
                hi[u] = tab[u] ? m.pois_off[l + 1] : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                jv[u] = 0;
                ry[u] = 0;
                ev[u] = 0;
                if (i0 + 64 * u < n) {
                    const r4 r = philox((uint32_t)v, (uint32_t)kk[u], t, TAG_PHI_CELL, m.key0, m.key1);
                    jv[u] = scale32(r.x, (uint32_t)(hi[u] - lo[u]));
                    ry[u] = r.y;
                    if (tab[u]) ev[u] = m.pois[lo[u] + jv[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (tab[u]) put(kk[u], (ry[u] < (uint32_t)ev[u]) ? (int32_t)jv[u] : (int32_t)(ev[u] >> 32));
                const uint64_t bal = __builtin_amdgcn_ballot_w64(past[u]);
                if (past[u]) lst[far + __builtin_popcountll(bal & below)] = (uint16_t)kk[u];
                far += __builtin_popcountll(bal);
            }
            lds_order();
        }
        // the others: rounded Gaussian of mean and variance lambda
        for (int32_t i0 = 0; i0 < far; i0 += 64) {
            if (i0 + lane < far) {
                const int32_t k = lst[i0 + lane];
                const r4 r = philox((uint32_t)v, (uint32_t)k, t, TAG_PHI_CELL, m.key0, m.key1);
                const double lam = tb + (double)g[k];
                const double rad = sqrt(-2.0 * log(1.0 - unit53(r.x, r.y)));
                const double gz = rad * cos(two_pi * unit53(r.z, r.w));
                const double y = floor(lam + sqrt(lam) * gz + 0.5);
                put(k, y > 0.0 ? (int32_t)y : 0);
            }
        }
        lds_order();

        long long pos_base = -1;
        for (uint32_t jb = 0;; jb += 64) {
            r4 r = philox((uint32_t)v, jb + (uint32_t)lane, t, TAG_PHI_PRIOR, m.key0, m.key1);
            const double e = -log(1.0 - unit53(r.x, r.y)) / bv;
            // a jump longer than K ends the column whatever its exact length
            const double capped = e < (double)K ? floor(e) : (double)K;
            const int32_t incl = group_scan_incl_i32<64>(1 + (int32_t)capped);
            const long long pos = pos_base + incl;
            if (pos < K) {
                int32_t *cell = &g[pos];
                int32_t x = 1;
                for (int q = 0; q < nT; ++q) x += (r.z >= T[q]) ? 1 : 0;
                const bool none = *cell == -1;
                if (none || vec) {
                    *cell = none ? x : *cell + x;
                    atomicAdd(&sum[pos], (unsigned long long)x);
                }
            }
            const long long last = pos_base + __builtin_amdgcn_readlane(incl, 63);
            if (last >= K) break;
            pos_base = last;
        }
        lds_order();

        // the word's largest draw and its nonzeros, then its row, four topics a lane
        int32_t cnt = 0, xmax = 0;
        for (int32_t k = 4 * lane; k < kpad; k += 256) {
            const int4 x = *(const int4 *)&g[k];
            cnt += (x.x > 0) + (x.y > 0) + (x.z > 0) + (x.w > 0);
            const int32_t a = x.x > x.y ? x.x : x.y, b = x.z > x.w ? x.z : x.w;
            const int32_t c = a > b ? a : b;
            xmax = c > xmax ? c : xmax;
        }
        const uint32_t fmt = __builtin_amdgcn_ballot_w64(xmax >= 0xFFFF) != 0
                                 ? ROW_32
                                 : (__builtin_amdgcn_ballot_w64(xmax > 0xFF) != 0 ? ROW_16 : ROW_8);
        auto row4 = [&](int32_t k) {
            const int4 x = *(const int4 *)&g[k];
            return make_uint4(x.x > 0 ? (uint32_t)x.x : 0u, x.y > 0 ? (uint32_t)x.y : 0u, x.z > 0 ? (uint32_t)x.z : 0u,
                              x.w > 0 ? (uint32_t)x.w : 0u);
        };
        if (fmt == ROW_8) {
            uint8_t *row = m.gam + draws_offset(m, ROW_8, v);
            for (int32_t k = 4 * lane; k < kpad; k += 256) {
                const uint4 x = row4(k);
                *(uint32_t *)(row + k) = x.x | x.y << 8 | x.z << 16 | x.w << 24;
            }
        } else if (fmt == ROW_16) {
            uint8_t *row = m.gam + draws_offset(m, ROW_16, v);
            for (int32_t k = 4 * lane; k < kpad; k += 256) {
                const uint4 x = row4(k);
                *(uint2 *)(row + 2 * k) = make_uint2(x.x | x.y << 16, x.z | x.w << 16);
            }
        } else {
            int32_t *row = (int32_t *)(m.gam + draws_offset(m, ROW_32, v));
            for (int32_t k = lane; k < K; k += 64) row[k] = g[k] > 0 ? g[k] : 0;
        }
        cnt = group_scan_incl_i32<64>(cnt);
        if (lane == 63) {
            m.colcnt[v] = cnt;
            m.phimax[v] = fmt << 30;
        }
        lds_order();
    }
    __syncthreads();
    for (int32_t k = threadIdx.x; k < K; k += 64 * WAVES) part[(int64_t)blockIdx.x * K + k] = sum[k];
}

// ---------------------------------------------------------------------------
// Phi-step, part 2: the first sum_blocks' worth of blocks after the scan's add
// the rows of partial sums (16 topics each, 64 threads to a topic): S_k, 1 /
// S_k and the empty topics.  The scan's blocks (the first) turn the columns'
// nonzeros into offsets: each adds up all columns before its own by itself,
// from L2 (V/2 counts on average), which takes one launch instead of three.
// Past COLS_BLOCKS tiles, where that costs more than another launch, one before
// sums each tile up: V = 200,000 11 us instead of 21, 2M 16 instead of 184, 16M
// 69 instead of 1,813.  It also lists the columns with more than ALIAS_SMALL
// nonzeros, in order.
// ---------------------------------------------------------------------------
constexpr int32_t ALIAS_SMALL = 256;
constexpr int32_t COLS_TILE = 4096;    // columns of a block, four a thread
constexpr int32_t COLS_BLOCKS = 16;    // most blocks that add up the columns before their own

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long x)
{
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// a column's nonzeros in the low 32 bits (fewer than 2^31 in all), one for a
// long column in the high
__device__ __forceinline__ unsigned long long col_val(int32_t c)
{
    return (unsigned long long)(uint32_t)c | ((unsigned long long)(c > ALIAS_SMALL) << 32);
}

// sum of a tile's columns
__global__ void __launch_bounds__(1024) cols_tiles_kernel(DevModel m, unsigned long long *tiles)
{
    __shared__ unsigned long long red[16];
    const int32_t v = blockIdx.x * COLS_TILE + 4 * threadIdx.x;
    unsigned long long t = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) t += v + u < m.V ? col_val(m.colcnt[v + u]) : 0;
    t = wave_sum_u64(t);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int j = 1; j < 16; ++j) t += red[j];
        tiles[blockIdx.x] = t;
    }
}

// (tiles: the sums of the tiles, or null)
__global__ void __launch_bounds__(1024) phi_sums_kernel(DevModel m, int32_t scan_blocks, const unsigned long long *tiles,
                                                        const unsigned long long *part, int32_t rows,
                                                        unsigned long long *stats)
{
    __shared__ unsigned long long red[1024];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if ((int)blockIdx.x >= scan_blocks) {
        const int32_t k = ((int)blockIdx.x - scan_blocks) * 16 + (tid & 15);
        unsigned long long s = 0;
        if (k < m.K) {
            int32_t r = tid >> 4;
            for (; r + 192 < rows; r += 256) {
                unsigned long long x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = part[(int64_t)(r + 64 * u) * m.K + k];
                s += (x[0] + x[1]) + (x[2] + x[3]);
            }
            for (; r < rows; r += 64) s += part[(int64_t)r * m.K + k];
        }
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (lane < 16) red[w * 16 + lane] = s;
        __syncthreads();
        if (tid < 16 && k < m.K) {
            s = 0;
            for (int j = 0; j < 16; ++j) s += red[j * 16 + tid];
            m.S[k] = s;
            m.Rd[k] = s ? 1.0 / (double)s : 0.0;
            if (s == 0 && stats) atomicAdd(&stats[ST_EMPTY_ROWS], 1ull);
        }
        return;
    }
    const int32_t v0 = (int32_t)blockIdx.x * COLS_TILE;
    const int32_t v1 = v0 + COLS_TILE < m.V ? v0 + COLS_TILE : m.V;
    unsigned long long t = 0;
    if (tiles) {
        for (int32_t i = tid; i < (int32_t)blockIdx.x; i += 1024) t += tiles[i];
    } else {
        for (int32_t v = 4 * tid; v < v0; v += 4 * 1024) {
            const int4 c = *(const int4 *)&m.colcnt[v];   // (v0 is a multiple of four)
            t += (col_val(c.x) + col_val(c.y)) + (col_val(c.z) + col_val(c.w));
        }
    }
    t = wave_sum_u64(t);
    if (lane == 0) red[w] = t;
    __syncthreads();
    unsigned long long base = 0;
    for (int j = 0; j < 16; ++j) base += red[j];
    const int32_t v = v0 + 4 * tid;
    unsigned long long c[4], own = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        c[u] = v + u < v1 ? col_val(m.colcnt[v + u]) : 0;
        own += c[u];
    }
    unsigned long long incl = own;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    __syncthreads();
    if (lane == 63) red[w] = incl;
    __syncthreads();
    unsigned long long at = base + incl - own;
    for (int j = 0; j < 16; ++j) {
        at += j < w ? red[j] : 0;
        base += red[j];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (v + u < v1) {
            m.colptr[v + u] = (int32_t)(uint32_t)at;
            if (c[u] >> 32) m.longcol[at >> 32] = v + u;
        }
        at += c[u];
    }
    if (v1 == m.V && tid == 0) {
        m.colptr[m.V] = (int32_t)(uint32_t)base;
        m.longcol[m.V] = (int32_t)(base >> 32);
        if (stats) stats[ST_NNZ_PHI] = base & 0xFFFFFFFFull;
    }
}

// (rows of partial sums: none for Algorithm 1, which has its own sums)
static hipError_t launch_phi_sums(const DevModel &m, const unsigned long long *part, int32_t rows,
                                  unsigned long long *stats, hipStream_t s)
{
    const int32_t nb = (m.V + COLS_TILE - 1) / COLS_TILE;
    unsigned long long *tiles = nullptr;
    if (nb > COLS_BLOCKS) {
        tiles = (unsigned long long *)m.scratch;
        cols_tiles_kernel<<<nb, 1024, 0, s>>>(m, tiles);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    phi_sums_kernel<<<nb + (rows ? (m.K + 15) / 16 : 0), 1024, 0, s>>>(m, nb, tiles, part, rows, stats);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Algorithm 1's Phi: phi = fp32(gamma / S_k), quotient in fp64 of the Gamma
// draws gamd and the row sums Sd; a cell is nonzero when its fp32 phi is
// normal (>= 2^-126).  Writes phid and compacts each column into the CSC
// (one wave per column, no LDS, so many columns are in flight).
// ---------------------------------------------------------------------------
constexpr float FP32_MIN_NORMAL = 0x1p-126f;

__global__ void __launch_bounds__(256) phi_dense_kernel(DevModel m)
{
    const int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= m.V) return;
    const int lane = __lane_id();
    const int32_t K = m.K;
    const int32_t cb = m.colptr[v];
    const double *gdcol = m.gamd + (int64_t)v * K;
    float *pcol = m.phid + (int64_t)v * K;
    int32_t run = 0;
    float fmax = 0.0f;
    // the column's draws are read PB rounds of 64 cells at a time, so that
    // many loads are in flight before the rounds are processed in order
    constexpr int PB = 8;
    for (int32_t kb = 0; kb < K; kb += 64 * PB) {
        double gs[PB];
#pragma unroll
        for (int j = 0; j < PB; ++j) {
            const int32_t k = kb + 64 * j + lane;
            gs[j] = k < K ? gdcol[k] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < PB; ++j) {
            const int32_t k0 = kb + 64 * j;
            if (k0 >= K) break;
            const int32_t k = k0 + lane;
            float f = 0.0f;
            if (k < K && m.Sd[k] > 0.0) {
                f = (float)(gs[j] / m.Sd[k]);
                f = f >= FP32_MIN_NORMAL ? f : 0.0f;
            }
            if (k < K) pcol[k] = f;
            fmax = f > fmax ? f : fmax;
            const uint64_t bal = __builtin_amdgcn_ballot_w64(f > 0.0f);
            if (f > 0.0f) {
                const int32_t e = run + __builtin_popcountll(bal & ((1ull << lane) - 1ull));
                m.ctopic[cb + e] = (uint16_t)k;
                m.cphi[cb + e] = f;
            }
            run += __builtin_popcountll(bal);
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const float y = __shfl_xor(fmax, o, 64);
        fmax = y > fmax ? y : fmax;
    }
    if (lane == 0) m.phimax[v] = __float_as_uint(fmax);
}

// ---------------------------------------------------------------------------
// Phi-step, part 3: each column of the CSC and its alias table for the a-part
// (weights alpha_k phi_kv; Vose's construction with FIFO work lists in
// ascending order; sigma_a = ascending fp64 sum of the weights), and the
// word's record.  The urn's columns (DIR false) are read from the word's row
// and compacted in LDS, phi = fp32(gamma / S_k) with the quotient in fp64 on
// full waves of nonzeros; Algorithm 1's are in the CSC already.
// Columns with at most ALIAS_SMALL nonzeros: one wave per column, four per
// block (LDS of ALIAS_SMALL entries each); the others: one column at a time
// per block with K entries of LDS.  Per entry: a probability (fp64), a
// work-list entry (u16), its topic (u16) and a turn mark (u8), so that many
// columns' chains run on a CU at once.
// Bound by the chain of sums of lane 0 (695 VALU instructions for a column of
// 120 nonzeros).  At V = 141,000, K = 1000: 200 us (short columns) and 125 us
// (long), from 440 + 155 + 180 us when a pass of its own wrote 14 bytes a
// cell and every column was launched twice.  The long columns come from the
// list, as V blocks that mostly return at once cost more than their work.
// ---------------------------------------------------------------------------
constexpr size_t alias_entry_bytes(bool dir)
{
    return sizeof(double) + (dir ? 1 : 2) * sizeof(uint16_t) + sizeof(uint8_t);
}

// the nonzeros of a word's row in ascending order, draw << 32 | topic in
// out; four topics a lane, JB rounds of 256 topics in flight
template <uint32_t FMT>
__device__ __forceinline__ void compact_row(const DevModel &m, int32_t v, uint64_t *out)
{
    constexpr int JB = 4;
    const int lane = __lane_id();
    const uint8_t *row = m.gam + draws_offset(m, FMT, v);
    int32_t run = 0;
    for (int32_t kb = 0; kb < m.ks16; kb += 256 * JB) {
        uint32_t x[JB][4];
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            const int32_t k = kb + 256 * j + 4 * lane;
            const bool in = k < m.ks16;
            if (FMT == ROW_8) {
                const uint32_t y = in ? *(const uint32_t *)(row + k) : 0u;
#pragma unroll
                for (int u = 0; u < 4; ++u) x[j][u] = (y >> (8 * u)) & 0xFFu;
            } else if (FMT == ROW_16) {
                const uint2 y = in ? *(const uint2 *)(row + 2 * k) : make_uint2(0u, 0u);
                x[j][0] = y.x & 0xFFFFu;
                x[j][1] = y.x >> 16;
                x[j][2] = y.y & 0xFFFFu;
                x[j][3] = y.y >> 16;
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) x[j][u] = k + u < m.K ? ((const uint32_t *)row)[k + u] : 0u;
            }
        }
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            if (kb + 256 * j >= m.ks16) break;
            const int32_t k = kb + 256 * j + 4 * lane;
            const int32_t c = (x[j][0] != 0) + (x[j][1] != 0) + (x[j][2] != 0) + (x[j][3] != 0);
            const int32_t incl = group_scan_incl_i32<64>(c);
            int32_t at = run + incl - c;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (x[j][u]) out[at] = ((uint64_t)x[j][u] << 32) | (uint32_t)(k + u);
                at += x[j][u] != 0;
            }
            run += __builtin_amdgcn_readlane(incl, 63);
        }
    }
}

template <bool SMALL, bool DIR>
__device__ __forceinline__ void phi_column(const DevModel &m, double *alias_lds, int32_t v, int wave, int32_t kpad)
{
    const int lane = __lane_id();
    const int32_t cb = m.colptr[v];
    const int32_t nv = m.colptr[v + 1] - cb;
    if (SMALL && nv > ALIAS_SMALL) return;
    const uint32_t pm = m.phimax[v];   // row format in the top bits; DIR: the largest phi
    const uint32_t fmt = DIR ? ROW_32 : pm >> 30;
    if (nv == 0) {
        if (lane == 0) {
            m.sigma_a[v] = 0.0;
            m.wrec[v] = make_uint4((uint32_t)cb, fmt << 30, 0u, 0u);
        }
        return;
    }
    const int32_t cap = SMALL ? ALIAS_SMALL : kpad;
    // this wave's region: cap entries (cap is a multiple of 64, so every
    // region and array stays 8-byte aligned)
    double *pq = (double *)((uint8_t *)alias_lds + (size_t)wave * cap * alias_entry_bytes(DIR));
    uint16_t *lst = (uint16_t *)(pq + cap);   // small entries from the front, large ones from the back
    uint16_t *ctop = DIR ? m.ctopic + cb : lst + cap;                   // topic of entry e
    uint8_t *mark = (uint8_t *)(lst + cap + (DIR ? 0 : cap));           // 1 at the FIFO steps where the head turned small
    if constexpr (!DIR) {
        if (fmt == ROW_8) compact_row<ROW_8>(m, v, (uint64_t *)pq);
        else if (fmt == ROW_16) compact_row<ROW_16>(m, v, (uint64_t *)pq);
        else compact_row<ROW_32>(m, v, (uint64_t *)pq);
        lds_order();
    }
    float fmax = 0.0f;
    // entry e's weight; the first reader of an entry completes the CSC
    auto weight = [&](int32_t e) -> double {
        if constexpr (DIR) {
            return m.alpha[ctop[e]] * (double)m.cphi[cb + e];
        } else {
            const uint64_t xk = ((const uint64_t *)pq)[e];
            const int32_t k = (int32_t)(uint32_t)xk;
            const float f = (float)((double)(uint32_t)(xk >> 32) / (double)m.S[k]);
            fmax = f > fmax ? f : fmax;
            ctop[e] = (uint16_t)k;
            m.ctopic[cb + e] = (uint16_t)k;
            m.cphi[cb + e] = f;
            return m.alpha[k] * (double)f;
        }
    };
    // weights w_e = alpha_k phi_kv in entry order (pq holds them first;
    // each lane also keeps its first MAXC chunks' weights in registers, all
    // chunks' loads issued together)
    constexpr int MAXC = SMALL ? ALIAS_SMALL / 64 : 16;
    double wr[MAXC];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int32_t e = c * 64 + lane;
        wr[c] = 0.0;
        if (e < nv) {
            wr[c] = weight(e);
            pq[e] = wr[c];
        }
    }
    for (int32_t e = MAXC * 64 + lane; e < nv; e += 64) pq[e] = weight(e);
    for (int32_t e = lane; e < nv; e += 64) mark[e] = 0;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // sigma_a: the ascending sum, read eight entries at a time
    double s = 0.0;
    if (lane == 0) {
        int32_t e = 0;
        for (; e + 8 <= nv; e += 8) {
            double b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) b[u] = pq[e + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += b[u];
        }
        for (; e < nv; ++e) s += pq[e];
        m.sigma_a[v] = s;
    }
    const double W = __shfl(s, 0, 64);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // p_e = w_e nv / W (w_e from registers: pq is reused); small
    // entries (p < 1) go to the front of lst in ascending order, large ones
    // to the back, the first large entry last; pq follows lst
    int32_t ns = 0, nl = 0;
    auto classify = [&](int32_t e, double w) {
        double p = 0.0;
        bool is_small = false;
        if (e < nv) {
            p = (w * (double)nv) / W;
            is_small = p < 1.0;
        }
        const uint64_t bs = __builtin_amdgcn_ballot_w64(e < nv && is_small);
        const uint64_t bl = __builtin_amdgcn_ballot_w64(e < nv && !is_small);
        const uint64_t below = (1ull << lane) - 1ull;
        if (e < nv) {
            const int32_t at = is_small ? ns + __builtin_popcountll(bs & below)
                                        : nv - 1 - (nl + __builtin_popcountll(bl & below));
            lst[at] = (uint16_t)e;
            pq[at] = p;
        }
        ns += __builtin_popcountll(bs);
        nl += __builtin_popcountll(bl);
    };
#pragma unroll
    for (int c = 0; c < MAXC; ++c)
        if (c * 64 < nv) classify(c * 64 + lane, wr[c]);
    // chunks past MAXC (K > 64 MAXC) recompute their weights
    for (int32_t e0 = MAXC * 64; e0 < nv; e0 += 64) {
        const int32_t e = e0 + lane;
        classify(e, e < nv ? m.alpha[ctop[e]] * (double)m.cphi[cb + e] : 0.0);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // Vose's pairing.  The FIFO of small entries is the initial small list
    // followed by large entries in the order they turn small, and a large
    // entry can only turn small at the head of the large list, so both lists
    // are walked with one index each.  FIFO step f pairs small entry sm(f),
    // of probability ps(f), with the head of the large list: its threshold is
    // floor(ps(f) 2^32), its alias the large entry at the head, and the
    // head's probability becomes (pg + ps(f)) - 1; below 1 the head turns
    // small (its residual joins the FIFO) and the next large entry leads.
    // Only that chain of sums is sequential: lane 0 runs it and marks the
    // steps at which the head turned small (its residual goes to its own pq
    // slot); then all lanes write the records, the head at step f being
    // large entry number sum_{f' < f} mark[f'] (a prefix sum over the wave).
    int32_t nf = 0;
    if (lane == 0) {
        int32_t gi = 0, f = 0;
        double pg = nl > 0 ? pq[nv - 1] : 0.0;
        auto step = [&](double ps) {
            pg = (pg + ps) - 1.0;
            if (pg < 1.0) {
                pq[nv - 1 - gi] = pg;
                mark[f] = 1;
                ++gi;
                if (gi < nl) pg = pq[nv - 1 - gi];
            }
            ++f;
        };
        // the initial small entries, read eight at a time
        for (int32_t i = 0; i < ns && gi < nl; i += 8) {
            double pb[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) pb[u] = pq[i + u < ns ? i + u : ns - 1];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + u < ns && gi < nl) step(pb[u]);
        }
        // then the large entries that turned small, in that order
        while (gi < nl && f - ns < gi) step(pq[nv - 1 - (f - ns)]);
        nf = f;
    }
    nf = __shfl(nf, 0, 64);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // each entry's record: thr | topic << 32 | alias topic << 48.  The FIFO's
    // first nf entries are paired (threshold floor(ps 2^32), alias the head
    // at their step); the others keep themselves (threshold 2^32 - 1)
    uint64_t *rec = m.calias + cb;
    int32_t heads = 0;   // turns before this chunk of steps
    for (int32_t f0 = 0; f0 < nf; f0 += 64) {
        const int32_t f = f0 + lane;
        const int32_t mk = f < nf ? mark[f] : 0;
        const int32_t incl = group_scan_incl_i32<64>(mk);
        if (f < nf) {
            const int32_t at = f < ns ? f : nv - 1 - (f - ns);
            const int32_t sm = lst[at];
            const double ps = pq[at];
            const int32_t head = heads + incl - mk;
            const uint32_t al = lst[nv - 1 - head];
            rec[sm] = (uint64_t)(uint32_t)floor(ps * 4294967296.0) | ((uint64_t)ctop[sm] << 32) |
                      ((uint64_t)ctop[al] << 48);
        }
        heads += __builtin_amdgcn_readlane(incl, 63);
    }
    for (int32_t i = (nf < ns ? nf : ns) + lane; i < ns; i += 64) {
        const uint64_t k = ctop[lst[i]];
        rec[lst[i]] = 0xFFFFFFFFull | (k << 32) | (k << 48);
    }
    for (int32_t j = (nf > ns ? nf - ns : 0) + lane; j < nl; j += 64) {
        const int32_t sm = lst[nv - 1 - j];
        const uint64_t k = ctop[sm];
        rec[sm] = 0xFFFFFFFFull | (k << 32) | (k << 48);
    }
    if constexpr (!DIR) {
        for (int o = 32; o > 0; o >>= 1) {
            const float y = __shfl_xor(fmax, o, 64);
            fmax = y > fmax ? y : fmax;
        }
    }
    if (lane == 0)
        m.wrec[v] = make_uint4((uint32_t)cb, (uint32_t)nv | fmt << 30, __float_as_uint((float)s),
                               DIR ? pm : __float_as_uint(fmax));
    lds_order();
}

template <bool SMALL, bool DIR>
__global__ void __launch_bounds__(SMALL ? 256 : 64) phi_alias_kernel(DevModel m)
{
    extern __shared__ double alias_lds[];
    if constexpr (SMALL) {
        const int wave = threadIdx.x >> 6;
        const int32_t v = blockIdx.x * 4 + wave;
        if (v < m.V) phi_column<true, DIR>(m, alias_lds, v, wave, 0);
    } else {
        const int32_t n = m.longcol[m.V];
        for (int32_t i = blockIdx.x; i < n; i += gridDim.x)
            phi_column<false, DIR>(m, alias_lds, __builtin_amdgcn_readfirstlane(m.longcol[i]), 0, m.ks16);
    }
}

// (of a Phi loaded as values)
__global__ void word_records_kernel(DevModel m)
{
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= m.V) return;
    const int32_t cb = m.colptr[v];
    m.wrec[v] = make_uint4((uint32_t)cb, (uint32_t)(m.colptr[v + 1] - cb) | ROW_32 << 30,
                           __float_as_uint((float)m.sigma_a[v]), m.phimax[v]);
}

hipError_t launch_word_records(const DevModel &m, hipStream_t s)
{
    word_records_kernel<<<(m.V + 255) / 256, 256, 0, s>>>(m);
    return hipGetLastError();
}

// columns and their alias tables (dir: Algorithm 1's)
static hipError_t launch_phi_columns(const DevModel &m, bool dir, int32_t n_cu, hipStream_t s)
{
    const size_t lds = 4 * ALIAS_SMALL * alias_entry_bytes(dir);
    if (dir) phi_alias_kernel<true, true><<<(m.V + 3) / 4, 256, lds, s>>>(m);
    else phi_alias_kernel<true, false><<<(m.V + 3) / 4, 256, lds, s>>>(m);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || m.K <= ALIAS_SMALL) return e;
    // as many blocks as the device holds (their number of columns is known
    // on the device only)
    const size_t long_lds = (size_t)m.ks16 * alias_entry_bytes(dir);
    int64_t blocks = (int64_t)(n_cu > 0 ? n_cu : 1) * (int64_t)(LDS_BYTES / long_lds);
    if (blocks < 1) blocks = 1;
    if (blocks > m.V) blocks = m.V;
    if (dir) phi_alias_kernel<false, true><<<(unsigned)blocks, 64, long_lds, s>>>(m);
    else phi_alias_kernel<false, false><<<(unsigned)blocks, 64, long_lds, s>>>(m);
    return hipGetLastError();
}

hipError_t launch_phi_step(const DevModel &m, unsigned long long *stats, int32_t n_cu, hipStream_t s)
{
    // the partial sums use the alias records' space, written after them
    unsigned long long *part = (unsigned long long *)m.calias;
    // persistent blocks: one row of partial sums each (K up to 4096: 128 KB)
    constexpr int W = PHI_DRAW_WAVES;
    const size_t lds = (size_t)m.ks16 * (PHI_SUM_BYTES + PHI_WAVE_BYTES * W);
    const int64_t fit = (int64_t)(LDS_BYTES / lds), most = 32 / W;
    int64_t blocks = (int64_t)(n_cu > 0 ? n_cu : 1) * (fit < most ? fit : most);
    const int64_t need = ((int64_t)m.V + W - 1) / W;
    if (blocks > need) blocks = need;
    const int32_t rows = (int32_t)blocks;
    phi_draw_kernel<<<rows, 64 * W, lds, s>>>(m, part, stats);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_phi_sums(m, part, rows, stats, s);
    if (e != hipSuccess) return e;
    return launch_phi_columns(m, false, n_cu, s);
}

// ---------------------------------------------------------------------------
// Algorithm 1's Phi-step: phi_k ~ Dir(n_k + beta) for every topic row, by
// the Gamma representation of the Dirichlet (Section 3.3): gamma_kv ~
// G(beta + n_kv, 1) and phi_kv = gamma_kv / S_k with S_k = sum_v gamma_kv.
// Gamma draws by Marsaglia and Tsang's method, which Section 3.4 names: for
// shape a >= 1, d = a - 1/3 and c = 1 / sqrt(9 d), a normal x gives
// t = 1 + c x (rejected when t <= 0) and v = t^3, kept as d v when a
// uniform u passes their squeeze u < 1 - 0.0331 x^4 or
// log u < x^2 / 2 + d (1 - v + log v); shapes below 1 use their boost
// G(a) = G(a + 1) U^(1/a), U^(1/a) taken as exp(log(U) / a).
// Attempt j of cell (k, v) at sweep t reads Philox counter
// (v, k, t, TAG_PHI_GAMMA + 256 j): the normal is Box-Muller's
// sqrt(-2 log u(r0)) cos(2 pi u(r1)), u = u(r2), and r3 of attempt 0 is the
// boost's U, with u(r) = (r + 1/2) 2^-32.  After 2^20 rejected attempts
// (probability below 0.05^(2^20)) the draw is d.
// ---------------------------------------------------------------------------
constexpr uint32_t GAMMA_TRIES = 1u << 20;

__device__ __forceinline__ double unit32o(uint32_t r) { return ((double)r + 0.5) * 0x1p-32; }

__device__ double gamma_draw(double a, uint32_t c0, uint32_t c1, uint32_t t, uint32_t key0, uint32_t key1)
{
    const double two_pi = 6.283185307179586476925286766559;
    const double a1 = a < 1.0 ? a + 1.0 : a;
    const double d = a1 - 1.0 / 3.0;
    const double c = 1.0 / sqrt(9.0 * d);
    double g = d;
    uint32_t boost = 0;
    for (uint32_t j = 0; j < GAMMA_TRIES; ++j) {
        const r4 r = philox(c0, c1, t, TAG_PHI_GAMMA + (j << 8), key0, key1);
        if (j == 0) boost = r.w;
        const double x = sqrt(-2.0 * log(unit32o(r.x))) * cos(two_pi * unit32o(r.y));
        const double t1 = 1.0 + c * x;
        if (t1 <= 0.0) continue;
        const double v = t1 * t1 * t1;
        const double u = unit32o(r.z);
        const double x2 = x * x;
        if (u < 1.0 - 0.0331 * (x2 * x2) || log(u) < 0.5 * x2 + d * (1.0 - v + log(v))) {
            g = d * v;
            break;
        }
    }
    if (a < 1.0) g = g * exp(log(unit32o(boost)) / a);
    return g;
}

// one cell per thread, word-major (cell v * K + k)
__global__ void __launch_bounds__(256) gamma_kernel(DevModel m)
{
    const int64_t cell = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t cells = (int64_t)m.V * m.K;
    if (cell >= cells) return;
    const uint32_t t = *m.tptr;
    const int32_t v = (int32_t)(cell / m.K);
    const int32_t k = (int32_t)(cell - (int64_t)v * m.K);
    const double a = (m.beta_v ? m.beta_v[v] : m.beta) + (double)m.n[cell];
    m.gamd[cell] = gamma_draw(a, (uint32_t)v, (uint32_t)k, t, m.key0, m.key1);
}

// S_k in two fixed-order passes (so the Phi-step is deterministic): block
// (b, j) sums its ROWSUM_COLS words in ascending order for 256 topics, 16
// words' draws in flight, then the blocks' partial sums are added in ascending
// order, 8 in flight.  At V = 28,000 and K = 1000 (224 MB) the first pass took
// 424 us with every topic in one block and a load waited for per word, now 39.
__global__ void __launch_bounds__(256) dsum_part_kernel(DevModel m, unsigned long long *stats)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && stats) stats[ST_EMPTY_ROWS] = 0;
    const int32_t v0 = blockIdx.x * ROWSUM_COLS;
    const int32_t v1 = v0 + ROWSUM_COLS < m.V ? v0 + ROWSUM_COLS : m.V;
    const int32_t k = blockIdx.y * 256 + threadIdx.x;
    if (k >= m.K) return;
    constexpr int U = 16;
    double s = 0.0;
    int32_t v = v0;
    for (; v + U <= v1; v += U) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = m.gamd[(int64_t)(v + u) * m.K + k];
#pragma unroll
        for (int u = 0; u < U; ++u) s += x[u];
    }
    for (; v < v1; ++v) s += m.gamd[(int64_t)v * m.K + k];
    m.dpart[(int64_t)blockIdx.x * m.K + k] = s;
}

__global__ void dsum_final_kernel(DevModel m, int32_t nb, unsigned long long *stats)
{
    const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= m.K) return;
    constexpr int U = 8;
    double s = 0.0;
    int32_t b = 0;
    for (; b + U <= nb; b += U) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = m.dpart[(int64_t)(b + u) * m.K + k];
#pragma unroll
        for (int u = 0; u < U; ++u) s += x[u];
    }
    for (; b < nb; ++b) s += m.dpart[(int64_t)b * m.K + k];
    m.Sd[k] = s;
    m.Rd[k] = 0.0;
    if (s == 0.0 && stats) atomicAdd(&stats[ST_EMPTY_ROWS], 1ull);
}

// nonzeros of each column: cells whose fp32 phi is normal; one wave per word
__global__ void __launch_bounds__(256) dcount_kernel(DevModel m)
{
    const int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= m.V) return;
    const int lane = __lane_id();
    const double *gdcol = m.gamd + (int64_t)v * m.K;
    int32_t cnt = 0;
    for (int32_t k = lane; k < m.K; k += 64) {
        const double S = m.Sd[k];
        const float f = S > 0.0 ? (float)(gdcol[k] / S) : 0.0f;
        cnt += f >= FP32_MIN_NORMAL;
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if (lane == 0) m.colcnt[v] = cnt;
}

hipError_t launch_phi_step_dirichlet(const DevModel &m, unsigned long long *stats, int32_t n_cu, hipStream_t s)
{
    if (m.phi_method != 1) return hipErrorInvalidValue;
    const int64_t cells = (int64_t)m.V * m.K;
    gamma_kernel<<<(unsigned)((cells + 255) / 256), 256, 0, s>>>(m);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int32_t nb = (m.V + ROWSUM_COLS - 1) / ROWSUM_COLS;
    dsum_part_kernel<<<dim3(nb, (m.K + 255) / 256), 256, 0, s>>>(m, stats);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    dsum_final_kernel<<<(m.K + 63) / 64, 64, 0, s>>>(m, nb, stats);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    dcount_kernel<<<(m.V + 3) / 4, 256, 0, s>>>(m);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_phi_sums(m, nullptr, 0, stats, s);
    if (e != hipSuccess) return e;
    phi_dense_kernel<<<(m.V + 3) / 4, 256, 0, s>>>(m);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_phi_columns(m, true, n_cu, s);
}

// ---------------------------------------------------------------------------
// z-step (Section 3.5).  A group of G lanes (G = 8, 16, 32, 64) owns one
// document at a time and walks its tokens in stored order (sequential Gibbs
// within the document), a block of up to G tokens at a time (one per lane).
//
// Slots.  Before a block's draws its tokens are staged: a token's word record
// and alias entry are loaded and its a-part topic drawn, which depends on the
// word and the token's random numbers only.  The block's topics are then
// known: a draw either takes the staged a-part topic or one with a nonzero
// count.  So the document's topics with a nonzero count and the block's
// a-part topics, in ascending order, are laid out once per block: topic e of
// them is slot e, and lane g holds the SL slots [g SL, g SL + SL).  The
// layout stays fixed for the whole block (a topic whose count falls to zero
// keeps its slot with a zero b-term), which is what makes a draw short:
//   - a slot's gather offset and R_k stay in registers, and the draws
//     phi_kv ~ x_kv of a later token are gathered DEPTH draws ahead;
//   - m_d is the slots' counts (exact): under 64 lanes in LDS as fp32,
//     changed by one LDS add each way per token and read once per draw, SL per
//     lane; on 64 lanes in registers (draw_regs);
//   - no topic list is kept sorted between draws, and no lane's result is
//     broadcast: the lane whose slots hold the crossing adds the token to its
//     slot itself.
// A set bit per topic in the list (P) and the number of list entries before
// each chunk of 2^log_b topics (pre) give a topic's slot by a popcount.
// Between blocks the counts lie by topic in LDS (mt, 1 or 2 bytes each): a
// layout is then one pass over the topic bits (1,970 cycles at K = 1000;
// 7,250 when the counts had to move from the old slots to the new).
//
// A draw of token i, with m^{-i} (Section 3.5):
//   sigma_b = sum_k phi_kv m_k over the slots, a group prefix sum ordering
//   the lanes, so running sums ascend in k; u (sigma_a + sigma_b) < sigma_a
//   takes the a-part, else the first slot whose running sum passes
//   y = u (sigma_a + sigma_b) - sigma_a.
//
// The b-part in fp32, with a proof of exactness.  Every quantity is within a
// known relative error of its exact value: a term
// b~ = fp32(fp32(fp32(x) R~_k) m) (R~_k = fp32(R_k)) or fp32(phi m) is within
// 5.01 u of phi_kv m_k (u = 2^-24; phi_kv itself is rounded to fp32), a lane's running sum of SL terms adds (SL - 1) u, the group
// scan log2(G) u, the exclusive prefix and y minus it u each (relative to
// Z = sigma_a + sigma_b).  x = u0 Z and y = x - sigma_a are within
// (SL + 8 + log2 G) u Z, so every comparison of y with 0 or with a running sum
// errs by less than (3 SL + 2 log2 G + 16) u Z.  The decision is taken only
// when y lies farther than tol = (64 + 8 SL) u Z from the boundary it is
// compared with (more than twice that error); it is then the decision of
// exact arithmetic, which is also the fp64 path's.  Otherwise (a few draws in
// ten thousand) slots_draw_f64 decides in fp64.  So the result is the fp64 one bit
// for bit, whatever the split of the topics over lanes.
//
// A document whose topics could pass SLOTS_MAX slots a lane takes more lanes (in
// fold-in and held-out calls: one whose topics are likely to); on 64, where that
// needs K > 1024, its list turns dense once it is longer: slot = topic, and every
// draw sums the word's Phi column with the counts read by topic (draw_dense;
// draw_overflow on fewer lanes).
//
// What bounds it: the draws of a document are a serial chain (LDS add, LDS
// read, the scan, the decision), so a long document is bound by the chain's
// latency and a full chip by VALU issue: see the figures at z_step_kernel.
// ---------------------------------------------------------------------------
struct ZArgs {
    DevModel m;
    DevCorpus c;
    const WorkItem *items;
    int32_t n_items;
    SlotLds lds;               // one group's layout
    int32_t r_bytes;           // the block's copy of R_k, at the start of LDS
    int32_t n_hot;             // frequent words counted per block in LDS (0: none)
    int32_t hot_off;           // their counters' byte offset in LDS
    int32_t *queue;
    unsigned long long *stats;
    double *ll_doc;         // per-document log-joint terms (or null)
};

// one draw's inputs, staged in LDS in draw order; every lane of the group
// reads them with one broadcast load
struct alignas(16) DrawRec {
    uint32_t row;    // byte offset of the word's row from gam (phid for values)
    float u0;        // (r >> 8) 2^-24, exact
    float saf;       // fp32(sigma_a(v)); NaN when it is too small for fp32's normal
                     // range (no comparison holds: the fp64 path decides)
    uint32_t w;      // row format | lane of the token << 2 (127: no draw)
    __device__ uint32_t fmt() const { return w & 3u; }
    __device__ int lane() const { return (int)__builtin_amdgcn_ubfe(w, 2, 7); }
};

// a record without a draw: it reads the first word's row, and its sigma_a
// (far above any sigma_b) makes it an a-part of no lane
constexpr uint32_t REC_NONE = ROW_32 | 127u << 2;
constexpr float REC_NONE_SA = 1e30f;

// draw statistics of a lane's tokens
struct ZStat {
    unsigned long long j = 0, jb = 0;    // sum of J; over the tokens not decided at staging
    uint32_t a = 0, deg = 0, fb = 0;     // a-part draws, degenerate tokens, fp64 draws
};

template <int G>
constexpr int log2g()
{
    return G == 64 ? 6 : (G == 32 ? 5 : (G == 16 ? 4 : 3));
}

// Global reads take a 32-bit byte offset from the table's base (the plan
// keeps every table under 4 GiB), so each address is one 32-bit add.
template <typename T>
__device__ __forceinline__ T load_at(const T *base, uint32_t byte_off)
{
    return *(const T *)((const char *)base + byte_off);
}

struct __attribute__((packed, aligned(1))) Unaligned32 {
    uint32_t x;
};

__device__ __forceinline__ uint32_t load_u32_at(const void *base, uint32_t byte_off)
{
    return ((const Unaligned32 *)((const char *)base + byte_off))->x;
}

// byte offset of word v's row from gam (phid for values)
__device__ __forceinline__ uint32_t row_offset(const DevModel &M, uint32_t fmt, int32_t v)
{
    return M.values ? (uint32_t)v * (uint32_t)M.K * 4u : draws_offset(M, fmt, v);
}

// the bits of a gathered word that are the draw
__device__ __forceinline__ uint32_t row_mask(uint32_t fmt) { return 0xFFFFFFFFu >> (32u - (8u << fmt)); }

// phi of a slot (to rounding) from the gathered word
template <bool VALUES>
__device__ __forceinline__ float slot_phi(uint32_t x, uint32_t mask, float R)
{
    return VALUES ? __uint_as_float(x) : (float)(x & mask) * R;
}

__device__ __forceinline__ float lds_add(float *p, float x)
{
    return __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// the document a group is working on (all pointers in LDS)
struct SlotDoc {
    uint8_t *mt;      // counts by topic, 1 or 2 bytes each (wide); up to date between blocks
    float *ms;        // counts by slot during a block (groups under 64 lanes)
    DrawRec *tok;     // the block's draws, in order
    uint32_t *P;      // a bit per topic: in the list
    uint16_t *lst;    // topic of each slot
    uint16_t *pre;    // list entries before each chunk of topics
    uint16_t *out;    // [G] the new slots of the block's draws, in order
    int32_t L;        // slots in use (group-uniform)
    int32_t nz;       // topics with a nonzero count (group-uniform)
    bool wide;        // (uniform)
    bool dense;       // slot = topic
};

__device__ __forceinline__ SlotDoc slot_doc(uint8_t *base, const SlotLds &A)
{
    SlotDoc S;
    S.mt = base;
    S.ms = (float *)(base + A.o_ms);
    S.tok = (DrawRec *)(base + A.o_tok);
    S.P = (uint32_t *)(base + A.o_p);
    S.lst = (uint16_t *)(base + A.o_lst);
    S.pre = (uint16_t *)(base + A.o_pre);
    S.out = (uint16_t *)(base + A.o_out);
    S.L = 0;
    S.nz = 0;
    S.wide = A.wide != 0;
    S.dense = false;
    return S;
}

// the count of topic k
__device__ __forceinline__ uint32_t count_of(const SlotDoc &S, int32_t k)
{
    return S.wide ? (uint32_t)((const uint16_t *)S.mt)[k] : (uint32_t)S.mt[k];
}

__device__ __forceinline__ void set_count(const SlotDoc &S, int32_t k, uint32_t c)
{
    if (S.wide) ((uint16_t *)S.mt)[k] = (uint16_t)c;
    else S.mt[k] = (uint8_t)c;
}

// the list bits of chunk ch (topics [ch 2^log_b, (ch + 1) 2^log_b))
__device__ __forceinline__ uint32_t chunk_bits(const uint32_t *P, int32_t ch, int32_t log_b)
{
    const int32_t k0 = ch << log_b;
    const uint32_t w = P[k0 >> 5] >> (k0 & 31);
    return log_b == 5 ? w : w & ((1u << (1 << log_b)) - 1u);
}

// the slot of topic k (in the list)
__device__ __forceinline__ int32_t slot_of(const SlotDoc &S, const SlotLds &A, int32_t k)
{
    if (S.dense) return k;
    const uint32_t bits = chunk_bits(S.P, k >> A.log_b, A.log_b);
    return (int32_t)S.pre[k >> A.log_b] + __builtin_popcount(bits & ((1u << (k & ((1 << A.log_b) - 1))) - 1u));
}

__device__ __forceinline__ int32_t topic_of(const SlotDoc &S, int32_t slot) { return S.dense ? slot : S.lst[slot]; }

// a document's counts from its tokens' topics z[s, e): by topic, and the
// list's bits
template <int G, bool STATS>
__device__ __forceinline__ void slots_load(SlotDoc &S, const SlotLds &A, const uint16_t *z, int64_t s, int64_t e,
                                           int g)
{
    for (int32_t i = g; i < A.o_ms / 16; i += G) ((uint4 *)S.mt)[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int32_t w = g; w < A.p_words; w += G) S.P[w] = 0u;
    S.L = 0;
    S.nz = 0;
    S.dense = false;
    lds_order();
    uint32_t *m32 = (uint32_t *)S.mt;
#pragma unroll 4
    for (int64_t i = s + g; i < e; i += G) {
        const uint32_t k = z[i];
        if (S.wide) atomicAdd(&m32[k >> 1], 1u << 16 * (k & 1));
        else atomicAdd(&m32[k >> 2], 1u << 8 * (k & 3));
        atomicOr(&S.P[k >> 5], 1u << (k & 31));
    }
    lds_order();
    if constexpr (STATS) {
        int32_t c = 0;
        for (int32_t w = g; w < A.p_words; w += G) c += __builtin_popcount(S.P[w]);
        S.nz = group_bcast<G>(group_scan_incl_i32<G>(c), G - 1);
    }
}

// lay the slots out for a block: the topics with a nonzero count (their bits
// are set) and each marked lane's topic ka
template <int G, bool BIG>
__device__ __forceinline__ void slots_layout(SlotDoc &S, const SlotLds &A, int32_t K, bool mark, int32_t ka, int g)
{
    if (mark) atomicOr(&S.P[ka >> 5], 1u << (ka & 31));
    lds_order();
    // list entries of this lane's chunks, and before them
    const int32_t c0 = g * A.ch_lane;
    int32_t n = 0;
    uint32_t bits0 = 0;
    for (int32_t j = 0; j < A.ch_lane; ++j)
        if (c0 + j < A.chunks) {
            const uint32_t bits = chunk_bits(S.P, c0 + j, A.log_b);
            bits0 = j == 0 ? bits : bits0;
            n += __builtin_popcount(bits);
        }
    const int32_t incl = group_scan_incl_i32<G>(n);
    const int32_t L = group_bcast<G>(incl, G - 1);
    if (BIG && __builtin_amdgcn_ballot_w64(S.dense || L > SLOTS_MAX * G) != 0) {
        S.dense = true;
        S.L = K;
        return;
    }
    S.L = L;
    int32_t o = incl - n;
    for (int32_t j = 0; j < A.ch_lane; ++j) {
        if (c0 + j >= A.chunks) break;
        S.pre[c0 + j] = (uint16_t)o;
        uint32_t bits = j == 0 ? bits0 : chunk_bits(S.P, c0 + j, A.log_b);
        const int32_t k0 = (c0 + j) << A.log_b;
        while (bits) {
            S.lst[o++] = (uint16_t)(k0 + __builtin_ctz(bits));
            bits &= bits - 1;
        }
    }
    lds_order();
}

// counts of this lane's slots, at the start of a block, and back: a topic
// whose count is zero leaves the list.  Slots past the list stand for topic
// K, whose count is zero and whose place the table has.  (No branch: one on
// a lane's slot costs more than an access that changes nothing.)
template <int SL>
__device__ __forceinline__ void slots_counts(const SlotDoc &S, const uint32_t (&kk)[SL], int32_t e0, int32_t K,
                                             uint32_t (&c)[SL])
{
    uint32_t k[SL];
#pragma unroll
    for (int u = 0; u < SL; ++u) k[u] = e0 + u < S.L ? kk[u] : (uint32_t)K;
    if (S.wide) {
#pragma unroll
        for (int u = 0; u < SL; ++u) c[u] = ((const uint16_t *)S.mt)[k[u]];
    } else {
#pragma unroll
        for (int u = 0; u < SL; ++u) c[u] = S.mt[k[u]];
    }
}

template <int SL>
__device__ __forceinline__ void slots_store(const SlotDoc &S, const uint32_t (&topics)[SL], int32_t e0, int32_t K,
                                            const uint32_t (&c)[SL], bool drop)
{
    // (opaque to the compiler, which would otherwise keep the addresses of
    // slots_counts, or spill them, throughout the block's draws)
    uint32_t kk[SL];
    asm volatile("" : "+v"(e0));
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        kk[u] = topics[u];
        asm volatile("" : "+v"(kk[u]));
    }
    if (S.wide) {
#pragma unroll
        for (int u = 0; u < SL; ++u) ((uint16_t *)S.mt)[e0 + u < S.L ? kk[u] : (uint32_t)K] = (uint16_t)c[u];
    } else {
#pragma unroll
        for (int u = 0; u < SL; ++u) S.mt[e0 + u < S.L ? kk[u] : (uint32_t)K] = (uint8_t)c[u];
    }
    if (drop) {
#pragma unroll
        for (int u = 0; u < SL; ++u)
            atomicAnd(&S.P[kk[u] >> 5], e0 + u < S.L && c[u] == 0 ? ~(1u << (kk[u] & 31)) : 0xFFFFFFFFu);
    }
    lds_order();
}

// a token of the block as its lane holds it
struct LaneTok {
    int32_t v;          // word
    int32_t ka;         // the a-part's alias draw (the old topic for an empty column)
    int32_t kv;         // nonzeros in the word's column
    uint32_t row, fmt;  // as DrawRec
    float u0, saf;
    bool sure;          // the a-part is certain whatever the document's counts, or
                        // the column is empty: no draw
};

__device__ __forceinline__ LaneTok no_token() { return {0, 0, 0, 0u, 0u, 0.0f, 1.0f, true}; }

// stage the token at this lane from its word's record.  nd: tokens in the
// document's counts.  The a-part's draw from the word's alias table over
// alpha_k phi_kv: slot j = floor(r1 K_v / 2^32), kept when r2 < its
// threshold, else its alias (Section 3.5).  The b-terms sum to
// sigma_b = sum_k phi_kv m_k <= phimax(v) (nd - 1), so when
// u (sigma_a + phimax(v) (nd - 1)) < sigma_a the token takes the a-part
// whatever the counts: tested in fp32 with a margin of 2^-20 (each side
// rounds by less than 6 2^-24), so a token so decided has
// x < sigma_a (1 - 10 2^-24) exactly, far outside any rounding of the sums.
__device__ __forceinline__ LaneTok stage_token(const DevModel &M, int32_t v, int32_t kold, const r4 &r,
                                               const int32_t nd)
{
    const uint4 rec = M.wrec[v];
    LaneTok x;
    x.v = v;
    const uint32_t kv = rec.y & WREC_LOW;
    x.kv = (int32_t)kv;
    x.fmt = rec.y >> 30;
    x.row = row_offset(M, x.fmt, v);
    x.u0 = (float)(r.x >> 8) * 0x1p-24f;
    const float sa = __uint_as_float(rec.z);
    x.saf = sa > 0x1p-100f ? sa : __uint_as_float(0x7FC00000u);
    x.ka = kold;
    x.sure = true;
    if (kv > 0) {
        const uint32_t j = scale32(r.y, kv);
        const uint64_t a = M.calias[rec.x + j];
        x.ka = (int32_t)((r.z < (uint32_t)a) ? ((a >> 32) & 0xFFFFu) : (a >> 48));
        const float B = __uint_as_float(rec.w) * (float)(nd - 1);
        x.sure = nd > 0 && x.u0 * (sa + B) < sa * (1.0f - 0x1p-20f);
    }
    return x;
}

// the group's lane whose terms hold y: the first whose running sum (incl, of
// the lanes' sums p) passes it; none (rounding): the last with a positive
// term; -1: no positive term, the a-part is the whole law
template <int G>
__device__ __forceinline__ int crossing_lane(double incl, double p, double y)
{
    const uint64_t bal = group_ballot<G>(incl > y);
    if (bal) return __builtin_ctzll(bal);
    const uint64_t pos = group_ballot<G>(p > 0.0);
    return pos ? 63 - __builtin_clzll(pos) : -1;
}

// The draw in fp64 over the slots, `per` a lane: every lane sums its terms in
// ascending order, the group scan orders the lanes.  count(e, k): the count of
// slot e, of topic k.  Returns the slot of the new topic, or -1 for the
// a-part; Z: sigma_a + sigma_b.
template <int G, typename Count>
__device__ __forceinline__ int32_t slots_draw_f64(const DevModel &M, const SlotDoc &S, int32_t v, float u0, int32_t per,
                                                  Count count, double &Z)
{
    // (opaque, or each number of slots' addresses of this seldom taken path
    // are computed, and spilled, at the start of the kernel)
    int g = __lane_id() & (G - 1);
    asm volatile("" : "+v"(g));
    const int32_t e0 = g * per;
    const int32_t e1 = e0 + per < S.L ? e0 + per : S.L;
    // term of entry e (exact in fp64: a 24-bit phi times a count below 2^16;
    // none for a topic without a count, whatever its loaded phi)
    auto term = [&](int32_t e) -> double {
        const int32_t k = S.lst[e];
        const float f = phi_at(M, v, k);
        const uint32_t c = count(e, k);
        return c ? (double)f * (double)c : 0.0;
    };
    double p = 0.0;
#pragma unroll 1
    for (int32_t e = e0; e < e1; ++e) p += term(e);
    const double incl = group_scan_incl<G>(p);
    const double sa = M.sigma_a[v];
    Z = sa + group_bcast_f64<G>(incl, G - 1);
    const double x = (double)u0 * Z;
    if (x < sa) return -1;
    const double y = x - sa;
    const int f = crossing_lane<G>(incl, p, y);
    if (f < 0) return -1;
    int32_t at = -1;
    if (g == f) {
        double c = incl - p;
#pragma unroll 1
        for (int32_t e = e0; e < e1; ++e) {
            const double b = term(e);
            if (b > 0.0) {
                c += b;
                at = e;
                if (c > y) break;
            }
        }
    }
    return __shfl(at, f, G);
}

// a word's Phi column: its first CSC entry and their number
struct Column {
    uint32_t first;
    int32_t n;
};

__device__ __forceinline__ Column column_of(const DevModel &M, int32_t v)
{
    const uint4 rec = M.wrec[v];
    return {rec.x, (int32_t)(rec.y & WREC_LOW)};
}

// A column on G lanes: chunks of G N entries, N neighbours a lane, so that a chunk
// is a few contiguous loads; on 64 lanes N = COL_N (one chunk) for columns of up
// to 64 COL_N entries, COL_B for longer ones
constexpr int COL_N = 4, COL_B = COL_PAD;

template <int G>
__device__ __forceinline__ int32_t col_chunks(const Column &c) { return (c.n + G * COL_B - 1) / (G * COL_B); }

struct ColEntries {
    float f[COL_B];
    uint16_t k[COL_B];
};

// COL_B entries of a column from entry e on
__device__ __forceinline__ ColEntries col_entries(const DevModel &M, const Column &c, int32_t e)
{
    const uint32_t i = c.first + (uint32_t)(e < c.n ? e : c.n);
    ColEntries x;
    __builtin_memcpy(x.f, M.cphi + i, sizeof(x.f));
    __builtin_memcpy(x.k, M.ctopic + i, sizeof(x.k));
    return x;
}

// the count of topic k in the dense layout of 64 lanes (documents of 960 tokens
// and more: two bytes)
__device__ __forceinline__ uint32_t dense_count(const SlotDoc &S, int32_t k) { return ((const uint16_t *)S.mt)[k]; }

// The draw in fp64 over the word's column, the counts read by topic: the sum of
// its chunks, then once more up to the chunk that holds the crossing.  Returns
// the new topic, or -1 for the a-part.
template <int G>
__device__ __forceinline__ int32_t column_draw_f64(const DevModel &M, const SlotDoc &S, int32_t v, float u0, double &Z)
{
    int g = __lane_id() & (G - 1);
    asm volatile("" : "+v"(g));
    const Column col = column_of(M, v);
    const int32_t chunks = col_chunks<G>(col);
    ColEntries x = {};
    double b[COL_B], p = 0.0;
    auto terms = [&](int32_t ch) {
        x = col_entries(M, col, (ch * G + g) * COL_B);
        const int32_t own = col.n - (ch * G + g) * COL_B;
        p = 0.0;
#pragma unroll
        for (int u = 0; u < COL_B; ++u) {
            const uint32_t c = u < own ? (G == 64 ? dense_count(S, x.k[u]) : count_of(S, x.k[u])) : 0u;
            b[u] = c ? (double)x.f[u] * (double)c : 0.0;
            p += b[u];
        }
    };
    double T = 0.0;
#pragma unroll 1
    for (int32_t ch = 0; ch < chunks; ++ch) {
        terms(ch);
        T = group_bcast_f64<G>(T + group_scan_incl<G>(p), G - 1);
    }
    const double sa = M.sigma_a[v];
    Z = sa + T;
    const double xz = (double)u0 * Z;
    if (xz < sa) return -1;
    const double y = xz - sa;
    double before = 0.0;
    int32_t k = -1;      // (where rounding leaves no crossing: the last positive term)
#pragma unroll 1
    for (int32_t ch = 0; ch < chunks; ++ch) {
        terms(ch);
        const double incl = before + group_scan_incl<G>(p);
        const int f = crossing_lane<G>(incl, p, y);
        double c = incl - p;
        int32_t at = -1;
        bool found = false;
#pragma unroll
        for (int u = 0; u < COL_B; ++u) {
            if (b[u] > 0.0 && !found) {
                c += b[u];
                at = x.k[u];
                found = c > y;
            }
        }
        before = group_bcast_f64<G>(incl, G - 1);
        if (f >= 0) k = __shfl(at, f, G);
        if (before > y) break;
    }
    return k;
}

// a lane's token during a block: old slot, a-part slot, the counts its old
// and new slot held when it left and entered (for the statistics), and what
// was drawn
struct LaneDraw {
    int32_t po, pa;
    uint32_t key;       // segment << 7 | rank within it for a token decided at
                        // staging (segment: draws before it); ~0: none
    float ro, rn;       // (2 and 1: no topic left or entered)
    // counts in registers: topics with a nonzero count when the token was
    // moved, when the block's draw number g was drawn, and the draws that
    // took the a-part
    int32_t kd, kd_draw;
    uint64_t a_draws;
    uint32_t a, fb;
};

// tokens decided at staging that lie before draw i: old slot to a-part slot,
// one after the other
template <bool STATS>
__device__ __forceinline__ void move_segment(const SlotDoc &S, LaneDraw &d, uint32_t i)
{
    uint32_t t = i << 7;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(d.key == t) == 0, 1)) return;
    do {
        if (d.key == t) {
            const float ro = lds_add(&S.ms[d.po], -1.0f), rn = lds_add(&S.ms[d.pa], 1.0f);
            if (STATS) {
                d.ro = ro;
                d.rn = rn;
            }
        }
        ++t;
    } while (__builtin_amdgcn_ballot_w64(d.key == t) != 0);
}

// the block's draws, n_max of them (the largest group's), with SL slots per
// lane; DEPTH draws' gathers in flight
template <int G, int SL, bool STATS, bool VALUES>
__device__ __forceinline__ void draw_slots(const DevModel &M, const SlotDoc &S, const float *Rf, const int32_t v,
                                           LaneDraw &d, const uint32_t n_max, const int lane_g)
{
    constexpr int DEPTH = SL <= 6 ? 2 : 1;
    // (opaque to the compiler, which would otherwise compute every SL's slot
    // addresses ahead of the token loop and spill them)
    int g = lane_g;
    asm volatile("" : "+v"(g));
    uint32_t kk[SL];       // topic of each slot (slots past the list: the first's)
    float R[SL];
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        const int32_t e = g * SL + u;
        kk[u] = S.lst[e < S.L ? e : 0];
        R[u] = Rf[kk[u]];
    }
    {
        uint32_t c[SL];
        slots_counts(S, kk, g * SL, M.K, c);
#pragma unroll
        for (int u = 0; u < SL; ++u) S.ms[g * SL + u] = (float)c[u];
        lds_order();
    }
    DrawRec rec[DEPTH];
    uint32_t x[DEPTH][SL];
    // one unaligned 4-byte load a slot, whatever the row's format (no branch
    // that would make the loads wait where its sides meet)
    auto gather = [&](int b) {
#pragma unroll
        for (int u = 0; u < SL; ++u) x[b][u] = load_u32_at(VALUES ? (const void *)M.phid : (const void *)M.gam, (kk[u] << rec[b].fmt()) + rec[b].row);
    };
#pragma unroll
    for (int b = 0; b < DEPTH; ++b) {
        rec[b] = S.tok[b];
        gather(b);
        // (in this order: the first draw then waits for its own loads only)
        __builtin_amdgcn_sched_barrier(0);
    }
    const uint64_t here = __builtin_amdgcn_ballot_w64(true);
    for (uint32_t i0 = 0; i0 < n_max; i0 += DEPTH) {
#pragma unroll
        for (int b = 0; b < DEPTH; ++b) {
            // (past n_max: records without a draw.  No early exit: the paths
            // would meet at the loop's end and make its first draw wait for
            // every load)
            const uint32_t i = i0 + b;
            move_segment<STATS>(S, d, i);
            const float u0 = rec[b].u0, sa = rec[b].saf;
            const int c = rec[b].lane();
            // phi of the slots (to rounding), from the gathered draws
            float f[SL];
            const uint32_t low = row_mask(rec[b].fmt());
#pragma unroll
            for (int u = 0; u < SL; ++u) f[u] = slot_phi<VALUES>(x[b][u], low, R[u]);
            rec[b] = S.tok[i + DEPTH < G ? i + DEPTH : G];
            // m^{-i}
            if (g == c) {
                if (STATS) d.ro = lds_add(&S.ms[d.po], -1.0f);
                else (void)lds_add(&S.ms[d.po], -1.0f);
            }
            float m[SL];
#pragma unroll
            for (int u = 0; u < SL; ++u) m[u] = S.ms[g * SL + u];
            // (issued before the gather's record is waited for: one LDS round
            // trip, not two)
            __builtin_amdgcn_sched_barrier(0);
            gather(b);
            // running sums of the lane's terms
            float cs[SL];
            cs[0] = f[0] * m[0];
#pragma unroll
            for (int u = 1; u < SL; ++u) cs[u] = cs[u - 1] + f[u] * m[u];
            const float incl = group_scan_incl_f32<G>(cs[SL - 1]);
            const float T = group_last_f32<G>(incl);
            const float Z = sa + T;
            const float y = u0 * Z - sa;
            const float tol = Z * ((float)(64 + 8 * SL) * 0x1p-24f);
            const bool is_a = y < -tol;
            // y relative to the lane's slots; how far it is from every
            // boundary of them, negative outside
            const float yl = y - (incl - cs[SL - 1]);
            float near = fminf(yl, cs[SL - 1] - yl);
#pragma unroll
            for (int u = 0; u + 1 < SL; ++u) near = fminf(near, fabsf(cs[u] - yl));
            const bool mine = near > tol;
            const uint64_t in_a = __builtin_amdgcn_ballot_w64(is_a), in_b = __builtin_amdgcn_ballot_w64(mine);
            if (mine) {
                // this lane's slots hold the crossing
                int32_t at = 0;
#pragma unroll
                for (int u = 0; u + 1 < SL; ++u) at += cs[u] <= yl ? 1 : 0;
                at += g * SL;
                (void)lds_add(&S.ms[at], 1.0f);
                S.out[i] = (uint16_t)at;
            }
            if (is_a && g == c) {
                if (STATS) d.rn = lds_add(&S.ms[d.pa], 1.0f);
                else (void)lds_add(&S.ms[d.pa], 1.0f);
                d.a = 1;
            }
            // a decided group has all its lanes in in_a or one in in_b
            if (__builtin_expect(
                    __builtin_popcountll(in_a) + G * __builtin_popcountll(in_b) != __builtin_popcountll(here), 0)) {
                // (a record without a draw can only be open where loaded values pass fp32's range)
                const bool open = !is_a && group_ballot<G>(mine) == 0 && c < G;
                double Zd;
                const int32_t vc = __shfl(v, c & (G - 1), G);
                const int32_t at = slots_draw_f64<G>(
                    M, S, vc, u0, SL, [&](int32_t e, int32_t) { return (uint32_t)S.ms[e]; }, Zd);
                if (open) {
                    if (at >= 0) {
                        if (g == 0) {
                            (void)lds_add(&S.ms[at], 1.0f);
                            S.out[i] = (uint16_t)at;
                        }
                    } else if (g == c) {
                        const float was = lds_add(&S.ms[d.pa], 1.0f);
                        if (STATS) d.rn = was;
                        d.a = 1;
                    }
                    if (g == c) d.fb = 1;
                }
            }
        }
    }
    // the tokens behind the last draw (a step past n_max has moved them)
    if (n_max % DEPTH == 0) move_segment<STATS>(S, d, n_max);
    lds_order();
    uint32_t c[SL];
#pragma unroll
    for (int u = 0; u < SL; ++u) c[u] = (uint32_t)S.ms[g * SL + u];
    slots_store(S, kk, g * SL, M.K, c, true);
}

// The block's draws of one document per wave (64 lanes), the counts in
// registers too: lane g holds the counts of its SL slots for the whole block
// (written back to LDS at the end), one per register, or with BYTES (SL <= 4,
// no count above 255) one per byte of one register, where an addition needs
// no compare per slot.  A draw touches LDS for its record only, read DEPTH
// draws ahead, so its chain is the scan and the decision.  Control is
// uniform: draws and moves are bit masks over the block's tokens.
//
// A wave alone on its SIMD issues an instruction every 4 to 5 cycles, a
// taken branch costs 20 to 90 and a branch on a vector compare 33: so a draw
// is straight-line code (about 80 instructions at SL = 3), whichever part it
// takes, and what is seldom needed stands outside the loop: a round of DEPTH
// draws in which one is undecided in fp32 is taken back and drawn again up to
// that one in fp64.
struct alignas(16) RegRec {
    uint32_t row;       // as DrawRec
    float u0, saf;
    uint32_t w;         // bits of a draw in the row (8, 16; 31 stands for 32) | row format << 30
    uint32_t o, a;      // old and a-part slot; BYTES: the lane that holds it
    uint32_t io, ia;    // BYTES: 1 in its byte
};

constexpr int REG_PAD = 8;      // records past the block's draws that may be read
constexpr uint32_t REG_NONE = 0xFFFFu;   // no slot, no lane

template <int SL, bool STATS, bool VALUES, bool BYTES>
__device__ __forceinline__ void draw_regs(const DevModel &M, SlotDoc &S, const float *Rf, const LaneTok &t,
                                          const bool draw, const uint32_t place, uint64_t moves,
                                          const uint64_t move_draws, const uint32_t n_draws, LaneDraw &d,
                                          const int lane_g)
{
    static_assert(!BYTES || SL <= 4, "four counts a register");
    constexpr int DEPTH = SL <= 2 ? 4 : (SL <= 4 ? 3 : (SL <= 10 ? 2 : 1));
    constexpr int NM = BYTES ? 1 : SL;
    int g = lane_g;
    asm volatile("" : "+v"(g));
    const int32_t e0 = g * SL;
    RegRec *const recs = (RegRec *)S.tok;
    {
        RegRec r = {0u, 0.0f, REC_NONE_SA, 31u | ROW_32 << 30, REG_NONE, REG_NONE, 0u, 0u};
        if (g < REG_PAD) recs[64 + g] = r;
        if (draw) {
            r.row = t.row;
            r.u0 = t.u0;
            r.saf = t.saf;
            r.w = (t.fmt == ROW_32 ? 31u : 8u << t.fmt) | t.fmt << 30;
            if (BYTES) {
                r.o = (uint32_t)d.po / SL;
                r.a = (uint32_t)d.pa / SL;
                r.io = 1u << 8 * (d.po - (int32_t)r.o * SL);
                r.ia = 1u << 8 * (d.pa - (int32_t)r.a * SL);
            } else {
                r.o = (uint32_t)d.po;
                r.a = (uint32_t)d.pa;
            }
        }
        recs[place] = r;
    }
    uint32_t kk[SL];
    float R[SL];
    uint32_t m[NM];
    if (BYTES) m[0] = 0;
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        const int32_t e = e0 + u;
        kk[u] = S.lst[e < S.L ? e : 0];
        R[u] = VALUES ? 0.0f : Rf[kk[u]];
    }
    {
        uint32_t c[SL];
        slots_counts(S, kk, e0, M.K, c);
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            if (BYTES) m[0] |= c[u] << 8 * u;
            else m[BYTES ? 0 : u] = c[u];
        }
    }
    lds_order();
    // count of slot u, and in fp32
    auto at = [&](int u) { return BYTES ? (m[0] >> 8 * u) & 255u : m[BYTES ? 0 : u]; };
    // add (sign: 1 or -1) the token at slot e (a uniform slot number)
    auto add = [&](int32_t e, bool up) {
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            const uint32_t one = e - e0 == u ? 1u : 0u;
            if (BYTES) m[0] = up ? m[0] + (one << 8 * u) : m[0] - (one << 8 * u);
            else m[BYTES ? 0 : u] = up ? m[BYTES ? 0 : u] + one : m[BYTES ? 0 : u] - one;
        }
    };
    RegRec rec[DEPTH];
    uint32_t x[DEPTH][SL];
    auto gather = [&](int b) {
        const uint32_t fmt = rec[b].w >> 30;
#pragma unroll
        for (int u = 0; u < SL; ++u)
            x[b][u] = load_u32_at(VALUES ? (const void *)M.phid : (const void *)M.gam, (kk[u] << fmt) + rec[b].row);
    };
    // topics with a nonzero count
    auto count = [&]() {
        int32_t n = 0;
#pragma unroll
        for (int u = 0; u < SL; ++u) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(at(u) != 0));
        return n;
    };
    auto store = [&](bool drop) {
        uint32_t c[SL];
#pragma unroll
        for (int u = 0; u < SL; ++u) c[u] = at(u);
        slots_store(S, kk, e0, M.K, c, drop);
    };
    const uint32_t po_pa = (uint32_t)d.po | ((uint32_t)d.pa << 16);
    // (lane i: the token of draw i)
    const int32_t token = __builtin_amdgcn_ds_permute((int)place << 2, g);
    auto move_before = [&](uint64_t below) {
        uint64_t todo = moves & below;
        moves &= ~below;
        while (todo) {
            const int c = __builtin_ctzll(todo);
            todo &= todo - 1;
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)po_pa, c);
            add((int32_t)(w & 0xFFFFu), false);
            if constexpr (STATS) {
                const int32_t n = count();
                if (g == c) d.kd = n;
            }
            add((int32_t)(w >> 16), true);
        }
    };
    auto moves_of_draw = [&](uint32_t i) {
        move_before((1ull << __builtin_amdgcn_readlane(token, (int)i)) - 1ull);
    };
    uint64_t a_draws = 0;      // draws that took the a-part
    uint32_t start = 0;
    while (start < n_draws) {
        // Rounds of DEPTH draws, every step of them run also past the last
        // draw (those records change nothing): an exit inside a round would
        // meet the loop's end and make its first step wait for every load.
#pragma unroll
        for (int b = 0; b < DEPTH; ++b) {
            rec[b] = recs[start + b];
            gather(b);
            __builtin_amdgcn_sched_barrier(0);
        }
        uint32_t i0 = start, open = 0;
        uint64_t moves0 = moves;
        uint32_t m0[NM];
#pragma unroll
        for (int u = 0; u < NM; ++u) m0[u] = m[u];
        // places of the round's results, and this lane's for no result
        const uint32_t nowhere = 64u + (uint32_t)g;
        for (; i0 < n_draws; i0 += DEPTH) {
            const uint64_t mv = move_draws >> i0;
            open = 0;
            moves0 = moves;
#pragma unroll
            for (int u = 0; u < NM; ++u) m0[u] = m[u];
#pragma unroll
            for (int b = 0; b < DEPTH; ++b) {
                const uint32_t i = i0 + b;
                if (mv & (1ull << b)) moves_of_draw(i);
                const RegRec r = rec[b];
                float f[SL];
#pragma unroll
                for (int u = 0; u < SL; ++u)
                    f[u] = VALUES ? __uint_as_float(x[b][u]) : (float)__builtin_amdgcn_ubfe(x[b][u], 0u, r.w) * R[u];
                rec[b] = recs[i + DEPTH];
                // m^{-i}
                if (BYTES) {
                    m[0] -= (uint32_t)g == r.o ? r.io : 0u;
                } else {
                    const uint32_t ro = r.o - (uint32_t)e0;
#pragma unroll
                    for (int u = 0; u < NM; ++u) m[u] -= ro == (uint32_t)u ? 1u : 0u;
                }
                if constexpr (STATS) {
                    const int32_t n = count();
                    if ((uint32_t)g == i) d.kd_draw = n;
                }
                float cs[SL];
                cs[0] = f[0] * (float)at(0);
#pragma unroll
                for (int u = 1; u < SL; ++u) cs[u] = cs[u - 1] + f[u] * (float)at(u);
                const float incl = group_scan_incl_f32<64>(cs[SL - 1]);
                const float T = group_last_f32<64>(incl);
                gather(b);
                const float Z = r.saf + T;
                const float y = r.u0 * Z - r.saf;
                const float tol = Z * ((float)(64 + 8 * SL) * 0x1p-24f);
                const bool is_a = y < -tol;
                // y relative to the lane's slots; how far it is from every
                // boundary of them, negative outside; the first slot whose
                // running sum passes it
                const float yl = y - (incl - cs[SL - 1]);
                float near = fminf(yl, cs[SL - 1] - yl);
                uint32_t n = 0;
#pragma unroll
                for (int u = 0; u + 1 < SL; ++u) {
                    near = fminf(near, fabsf(cs[u] - yl));
                    n += cs[u] <= yl ? 1u : 0u;
                }
                const bool mine = near > tol;
                // the a-part's slot gains the token, or this lane's slot n
                if (BYTES) {
                    const uint32_t ga = (uint32_t)g == r.a ? r.ia : 0u;
                    const uint32_t gb = mine ? 1u << (8u * n) : 0u;
                    m[0] += is_a ? ga : gb;
                } else {
                    const uint32_t gain = is_a ? r.a - (uint32_t)e0 : (mine ? n : REG_NONE);
#pragma unroll
                    for (int u = 0; u < NM; ++u) m[u] += gain == (uint32_t)u ? 1u : 0u;
                }
                S.out[mine ? i : nowhere] = (uint16_t)((uint32_t)e0 + n);
                const uint64_t in_a = __builtin_amdgcn_ballot_w64(is_a), in_b = __builtin_amdgcn_ballot_w64(mine);
                open |= (in_a | in_b) == 0 ? 1u << b : 0u;
                if constexpr (STATS) a_draws |= in_a & (i < n_draws ? 1ull << i : 0ull);
            }
            if (__builtin_expect(open != 0, 0)) break;
        }
        // (a record past the last draw can only be open where loaded values
        // pass fp32's range)
        if (open) open &= (uint32_t)((2ull << (n_draws - 1 - i0)) - 1ull);
        if (__builtin_expect(open == 0, 1)) break;
        // a draw of this round is too close to a boundary for fp32: the round
        // again up to it, in fp64 from the counts in LDS (the draws before it
        // give what they gave)
        moves = moves0;
#pragma unroll
        for (int u = 0; u < NM; ++u) m[u] = m0[u];
        const uint32_t end = i0 + (uint32_t)__builtin_ctz(open) + 1;
        // (the draws behind it start over, as if not drawn: their places are
        // the a-part's again)
        a_draws &= (1ull << i0) - 1ull;
        if (place >= end && place < i0 + DEPTH) S.out[place] = (uint16_t)d.pa;
        for (uint32_t i = i0; i < end; ++i) {
            if ((move_draws >> i) & 1ull) moves_of_draw(i);
            const int c = __builtin_amdgcn_readlane(token, (int)i);
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)po_pa, c);
            add((int32_t)(w & 0xFFFFu), false);
            if constexpr (STATS) {
                const int32_t n = count();
                if ((uint32_t)g == i) d.kd_draw = n;
            }
            store(false);
            double Zd;
            int32_t to = slots_draw_f64<64>(
                M, S, __builtin_amdgcn_readlane(t.v, c), recs[i].u0, SL,
                [&](int32_t, int32_t k) { return count_of(S, k); }, Zd);
            lds_order();
            if (to < 0) {
                to = (int32_t)(w >> 16);
                a_draws |= 1ull << i;
            }
            if (g == 0) S.out[i] = (uint16_t)to;
            if (g == c && i + 1 == end) d.fb = 1;
            add(to, true);
            lds_order();
        }
        start = end;
    }
    move_before(~0ull);
    store(true);
    if constexpr (STATS) {
        S.nz = count();
        d.a_draws = a_draws;
    }
}

// The block's draws of lists that pass SLOTS_MAX slots a lane on fewer than 64
// lanes, slot = topic for every group of the wave: one fp64 draw over the word's
// column after the other.
template <int G>
__device__ __forceinline__ void draw_overflow(const DevModel &M, const SlotDoc &S, const int32_t v, const LaneDraw &d,
                                              const uint32_t n_max, const int g)
{
    auto change = [&](int32_t k, int by) { set_count(S, k, count_of(S, k) + (uint32_t)by); };
    auto moves = [&](uint32_t i) {
        for (uint32_t t = i << 7; __builtin_amdgcn_ballot_w64(d.key == t) != 0; ++t) {
            if (d.key == t) {
                change(d.po, -1);
                change(d.pa, 1);
            }
            lds_order();
        }
    };
#pragma unroll 1
    for (uint32_t i = 0; i < n_max; ++i) {
        moves(i);
        const DrawRec rec = S.tok[i];
        const int c = rec.lane();   // (127: the group has no draw left)
        if (g == c) change(d.po, -1);
        lds_order();
        double Z;
        const int32_t k = column_draw_f64<G>(M, S, __shfl(v, c & (G - 1), G), rec.u0, Z);
        if (g == c) {
            change(k >= 0 ? k : d.pa, 1);
            if (k >= 0) S.out[i] = (uint16_t)k;
        }
        lds_order();
    }
    moves(n_max);
}

// The terms of a lane's N entries of a column and their sum; own: how many of
// them are the column's (FULL: all)
template <int N, bool FULL>
__device__ __forceinline__ float col_terms(const SlotDoc &S, const ColEntries &x, int32_t own, int32_t K, float (&b)[N])
{
    uint32_t c[N];
#pragma unroll
    for (int u = 0; u < N; ++u) c[u] = dense_count(S, FULL || u < own ? x.k[u] : K);   // (topic K: no count)
    float p = 0.0f;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        b[u] = FULL || u < own ? x.f[u] * (float)c[u] : 0.0f;
        p += b[u];
    }
    return p;
}

// the topic of a lane's N entries that holds y, s the running sum before them;
// -2: none, or too close to a boundary
template <int N>
__device__ __forceinline__ int32_t col_walk(const ColEntries &x, const float (&b)[N], float s, float y, float tol)
{
    int32_t at = -2;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const float hi = s + b[u];
        if (b[u] > 0.0f && s <= y && hi > y) at = y - s > tol && hi - y > tol ? (int32_t)x.k[u] : -2;
        s = hi;
    }
    return at;
}

// The block's draws in the dense layout (64 lanes; topic lists past SLOTS_MAX
// slots a lane): each sums its word's column in fp32, the counts read by topic,
// and decides as the draws over slots do; undecided ones are drawn in fp64.
// Lane c keeps the running sum after chunk c, and the chunk that holds the
// crossing is read once more.  What a draw reads from memory does not depend on
// the draws before it, so the records of two words and the first entries of one
// are loaded ahead.
// tol: a chunk's running sum adds one rounding to the bound at the head of
// this section, with SL = COL_B.
template <bool STATS>
__device__ __forceinline__ void draw_dense(const DevModel &M, const SlotDoc &S, const LaneTok &t, LaneDraw &d,
                                           const uint32_t place, const uint32_t n_draws, const int g)
{
    // one token leaves or enters topic k (one lane); the count before
    auto change = [&](uint32_t k, uint32_t by) {
        const uint32_t shift = (k & 1u) << 4;
        const uint32_t was = atomicAdd((uint32_t *)S.mt + (k >> 1), by << shift);
        return STATS ? (float)__builtin_amdgcn_ubfe(was, shift, 16u) : 0.0f;
    };
    auto moves = [&](uint32_t i) {
        for (uint32_t key = i << 7; __builtin_amdgcn_ballot_w64(d.key == key) != 0; ++key) {
            if (d.key == key) {
                const float ro = change((uint32_t)d.po, 0xFFFFFFFFu), rn = change((uint32_t)d.pa, 1u);
                if (STATS) {
                    d.ro = ro;
                    d.rn = rn;
                }
            }
        }
    };
    // (lane i: the token of draw i)
    const int32_t token = __builtin_amdgcn_ds_permute((int)place << 2, g);
    auto column = [&](uint32_t i) {
        const int c = __builtin_amdgcn_readlane(token, (int)(i < n_draws ? i : 0u));
        return column_of(M, __builtin_amdgcn_readlane(t.v, c));
    };
    auto head = [&](const Column &c) { return col_entries(M, c, g * (c.n <= 64 * COL_N ? COL_N : COL_B)); };
    Column col = column(0), next = column(1);
    ColEntries x = head(col);
    for (uint32_t i = 0; i < n_draws; ++i) {
        const Column after = column(i + 2);
        const ColEntries xn = head(next);
        moves(i);
        const int c = __builtin_amdgcn_readlane(token, (int)i);
        if (g == c) {
            const float ro = change((uint32_t)d.po, 0xFFFFFFFFu);
            if (STATS) d.ro = ro;
        }
        const float u0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t.u0), c));
        const float sa = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t.saf), c));
        float y, tol;
        auto decide = [&](float T, int32_t chunks) {
            const float Z = sa + T;
            y = u0 * Z - sa;
            tol = Z * ((float)(128 + 8 * chunks) * 0x1p-24f);
            return __builtin_amdgcn_ballot_w64(y < -tol) != 0 ? -1 : -2;
        };
        int32_t k;   // the new topic; -1: the a-part, -2: undecided
        if (col.n <= 64 * COL_N) {
            float b[COL_N];
            const float p = col_terms<COL_N, false>(S, x, col.n - g * COL_N, M.K, b);
            const float incl = group_scan_incl_f32<64>(p);
            k = decide(group_last_f32<64>(incl), 1);
            const uint64_t lanes = __builtin_amdgcn_ballot_w64(incl > y && y > tol);
            const int32_t at = col_walk<COL_N>(x, b, incl - p, y, tol);
            if (lanes != 0) k = __builtin_amdgcn_readlane(at, __builtin_ctzll(lanes));
        } else {
            static_assert(4096 <= 64 * 64 * COL_B, "a lane per chunk");
            const int32_t chunks = col_chunks<64>(col);
            float b[COL_B], p = 0.0f, incl = 0.0f, T = 0.0f, ends = 0.0f;
            int32_t ch = 0;
            auto add = [&] {
                incl = T + group_scan_incl_f32<64>(p);
                T = group_last_f32<64>(incl);
                ends = g == ch ? T : ends;
            };
            for (; ch + 1 < chunks; ++ch) {
                const ColEntries ahead = col_entries(M, col, ((ch + 1) * 64 + g) * COL_B);
                p = col_terms<COL_B, true>(S, x, 0, M.K, b);
                add();
                x = ahead;
            }
            p = col_terms<COL_B, false>(S, x, col.n - (ch * 64 + g) * COL_B, M.K, b);
            add();
            k = decide(T, chunks);
            const uint64_t over = __builtin_amdgcn_ballot_w64(g < chunks && ends > y && y > tol);
            if (over != 0) {
                ch = __builtin_ctzll(over);
                if (ch + 1 < chunks) {
                    x = col_entries(M, col, (ch * 64 + g) * COL_B);
                    p = col_terms<COL_B, true>(S, x, 0, M.K, b);
                    incl = group_scan_incl_f32<64>(p);
                    if (ch) incl += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ends), ch - 1));
                }
                const uint64_t lanes = __builtin_amdgcn_ballot_w64(incl > y);
                const int32_t at = col_walk<COL_B>(x, b, incl - p, y, tol);
                if (lanes != 0) k = __builtin_amdgcn_readlane(at, __builtin_ctzll(lanes));
            }
        }
        if (__builtin_expect(k == -2, 0)) {
            double Zd;
            k = column_draw_f64<64>(M, S, __builtin_amdgcn_readlane(t.v, c), u0, Zd);
            if (g == c) d.fb = 1;
        }
        if (g == c) {
            const float rn = change(k >= 0 ? (uint32_t)k : (uint32_t)d.pa, 1u);
            if (STATS) d.rn = rn;
            if (k >= 0) S.out[i] = (uint16_t)k;
            else d.a = 1;
        }
        lds_order();
        col = next;
        next = after;
        x = xn;
    }
    moves(n_draws);
}

// the block's records, in draw order, the lanes without a draw behind them
template <int G>
__device__ __forceinline__ void stage_draws(const SlotDoc &S, const LaneTok &x, const LaneDraw &d, bool draw,
                                            uint32_t place, int g)
{
    DrawRec rec;
    rec.row = draw ? x.row : 0u;
    rec.u0 = draw ? x.u0 : 0.0f;
    rec.saf = draw ? x.saf : REC_NONE_SA;
    rec.w = draw ? (x.fmt | ((uint32_t)g << 2)) : REC_NONE;
    S.tok[place] = rec;
    if (g < 2) {
        DrawRec none = {0u, 0.0f, REC_NONE_SA, REC_NONE};
        S.tok[G + g] = none;
    }
    lds_order();
}

// Draw a block of tokens, lane g's token x of old topic kold (valid: the
// lane has one), after slots_layout (bytes: no count can pass
// 255); returns the lane's new topic.  The
// group's lanes are converged.
template <int G, bool STATS, bool BIG>
__device__ __forceinline__ int32_t draw_block(const DevModel &M, SlotDoc &S, const SlotLds &A, const float *Rf,
                                              const LaneTok &x, int32_t kold, bool valid, bool bytes, ZStat &st,
                                              const int g)
{
    const bool draws = valid && !x.sure;
    const uint64_t db = group_ballot<G>(draws);
    const uint64_t below = (1ull << g) - 1ull;
    const uint32_t before = (uint32_t)__builtin_popcountll(db & below);
    const uint32_t nd = (uint32_t)__builtin_popcountll(db);
    LaneDraw d;
    d.po = valid ? slot_of(S, A, kold) : 0;
    d.pa = valid ? slot_of(S, A, x.ka) : 0;
    d.key = 0xFFFFFFFFu;
    const bool moves = valid && x.sure && x.kv > 0;
    // rank among the segment's tokens decided at staging (tokens of an empty
    // column keep their topic: no move)
    const uint64_t mb = group_ballot<G>(moves);
    const uint64_t prev = db & below;
    const uint64_t seg = prev ? below & ~((2ull << (63 - __builtin_clzll(prev))) - 1ull) : below;
    if (moves) d.key = (before << 7) | (uint32_t)__builtin_popcountll(mb & seg);
    d.ro = 2.0f;
    d.rn = 1.0f;
    d.kd = 0;
    d.kd_draw = 0;
    d.a_draws = 0;
    d.a = moves ? 1u : 0u;
    d.fb = 0;
    // draws in order, the lanes without one behind them; the drawn slots'
    // places start as the a-part's
    const uint32_t place = draws ? before : nd + (uint32_t)g - before;
    S.out[place] = (uint16_t)d.pa;
    lds_order();
    // the wave's largest number of draws (scalar: the ballot's fields)
    const uint64_t all = __builtin_amdgcn_ballot_w64(draws);
    uint32_t n_max = 0;
#pragma unroll
    for (int o = 0; o < 64; o += G) {
        const uint32_t n = (uint32_t)__builtin_popcountll(G == 64 ? all : (all >> o) & ((1ull << (G & 63)) - 1ull));
        n_max = n > n_max ? n : n_max;
    }
    auto over = [&](int sl) { return __builtin_amdgcn_ballot_w64(S.L > sl * G) != 0; };
    // (64 lanes: the draws that have moves before them, in draw order)
    uint64_t mv_draws = 0;
    if constexpr (G == 64) {
        const int first = draws && (mb & seg) != 0 ? 1 : 0;
        mv_draws = __builtin_amdgcn_ballot_w64(__builtin_amdgcn_ds_permute((int)place << 2, first) != 0);
    }
    bool regs = false;
#define PULDA_REGS(SL_, V_, B_) draw_regs<SL_, STATS, V_, B_>(M, S, Rf, x, draws, place, mb, mv_draws, nd, d, g)
#define PULDA_DRAW(SL_)                                                                            \
    do {                                                                                           \
        if constexpr (G == 64) {                                                \
            if (SL_ <= 4 && bytes) {                                                               \
                if (M.values) PULDA_REGS(SL_, true, SL_ <= 4);                                     \
                else PULDA_REGS(SL_, false, SL_ <= 4);                                             \
            } else {                                                                               \
                if (M.values) PULDA_REGS(SL_, true, false);                                        \
                else PULDA_REGS(SL_, false, false);                                                \
            }                                                                                      \
            regs = true;                                                                           \
        } else {                                                                                   \
            stage_draws<G>(S, x, d, draws, place, g);                                              \
            if (M.values) draw_slots<G, SL_, STATS, true>(M, S, Rf, x.v, d, n_max, g);             \
            else draw_slots<G, SL_, STATS, false>(M, S, Rf, x.v, d, n_max, g);                     \
        }                                                                                          \
    } while (0)
    if (!over(1)) PULDA_DRAW(1);
    else if (!over(2)) PULDA_DRAW(2);
    else if (!over(3)) PULDA_DRAW(3);
    else if (!over(4)) PULDA_DRAW(4);
    else if (!over(5)) PULDA_DRAW(5);
    else if (!BIG || !over(6)) PULDA_DRAW(6);
    else if constexpr (BIG) {
        if (!over(8)) PULDA_DRAW(8);
        else if (!over(10)) PULDA_DRAW(10);
        else if (!over(12)) PULDA_DRAW(12);
        else if (!S.dense) PULDA_DRAW(16);
        else if constexpr (G == 64) {
            draw_dense<STATS>(M, S, x, d, place, nd, g);
        } else if constexpr (!STATS) {   // (the z-step's documents fit)
            stage_draws<G>(S, x, d, draws, place, g);
            draw_overflow<G>(M, S, x.v, d, n_max, g);
        }
    }
#undef PULDA_DRAW
#undef PULDA_REGS
    lds_order();
    if constexpr (STATS) {
        // J = min(K_d^{-i}, K_v): the topics with a nonzero count when token
        // g was drawn, from the topics that left and entered before it
        int32_t Kd;
        if (regs) {
            const int32_t drawn = __shfl(d.kd_draw, (int)before, 64);
            Kd = draws ? drawn : d.kd;
            if (draws) d.a = (uint32_t)((d.a_draws >> before) & 1ull);
        } else {
            const int32_t left = d.ro == 1.0f ? 1 : 0;
            const int32_t delta = (d.rn == 0.0f ? 1 : 0) - left;
            const int32_t incl = group_scan_incl_i32<G>(delta);
            Kd = S.nz + incl - delta - left;
            S.nz += group_bcast<G>(incl, G - 1);
        }
        if (valid && x.kv > 0) {
            const uint32_t j = (uint32_t)(Kd < x.kv ? Kd : x.kv);
            st.j += j;
            if (draws) st.jb += j;
        }
        st.a += d.a;
        st.fb += d.fb;
        st.deg += valid && x.kv == 0 ? 1u : 0u;
    }
    return valid ? topic_of(S, draws ? S.out[place] : d.pa) : 0;
}

// HOT: the frequent words' count increments go to the block's counters in
// LDS (hist), the others' to n
template <int G, bool BIG, bool HOT>
__device__ __forceinline__ void z_step_item(const ZArgs &a, const WorkItem &w, const float *R, uint8_t *base,
                                            ZStat &st, uint32_t *hist)
{
    constexpr int NG = 64 / G;
    const int lane = __lane_id();
    const int g = lane & (G - 1);
    const int grp = lane / G;
    const SlotLds &A = a.lds;
    SlotDoc S = slot_doc(base + grp * A.group_bytes, A);
    const DevModel &M = a.m;
    const uint32_t t = *M.tptr;
    for (int32_t di = grp; di < w.count; di += NG) {
        const int32_t d = a.c.doc_order[w.first + di];
        const int64_t s = a.c.doc_off[d], e = a.c.doc_off[d + 1];
        if (s == e) {
            if (a.ll_doc && g == 0) a.ll_doc[d] = 0.0;
            continue;
        }
        slots_load<G, true>(S, A, a.c.z, s, e, g);
        for (int64_t i0 = s; i0 < e; i0 += G) {
            const int64_t i = i0 + g;
            const bool valid = i < e;
            int32_t zo = 0, wv = 0;
            LaneTok x = no_token();
            if (valid) {
                // the token stream is read once per sweep: non-temporal, so
                // it does not displace the tables that the draws reuse
                wv = __builtin_nontemporal_load(a.c.words + i);
                zo = __builtin_nontemporal_load(a.c.z + i);
                const r4 r = philox((uint32_t)i, (uint32_t)((uint64_t)i >> 32), t, TAG_Z, M.key0, M.key1);
                x = stage_token(M, wv, zo, r, (int32_t)(e - s));
            }
            slots_layout<G, BIG>(S, A, M.K, valid, x.ka, g);
            const int32_t znew = draw_block<G, true, BIG>(M, S, A, R, x, zo, valid, e - s < 256, st, g);
            // the count rebuild: each lane adds its own token, once the
            // block's draws are done (a frequent word's into the block's
            // counters in LDS, added to n when the kernel ends)
            if (valid) {
                __builtin_nontemporal_store((uint16_t)znew, a.c.z + i);
                const int32_t h = HOT ? M.hot[wv] : -1;
                if (HOT && h >= 0) atomicAdd(&hist[(uint32_t)h * (uint32_t)M.K + (uint32_t)znew], 1u);
                else atomicAdd(&M.n[(uint32_t)wv * (uint32_t)M.K + (uint32_t)znew], 1);
            }
        }
        if (a.ll_doc) {
            // the document's term of log p(z | alpha) for its final counts:
            // lgamma(A) - lgamma(N_d + A) + sum_k [lgamma(m_k + alpha) - lgamma(alpha)]
            double part = 0.0;
            for (int32_t j = g; j < S.L; j += G) part += M.lg_alpha[count_of(S, topic_of(S, j))];
            const double tot = group_bcast_f64<G>(group_scan_incl<G>(part), G - 1);
            if (g == 0) a.ll_doc[d] = tot + M.lg_A[e - s];
        }
        lds_order();
    }
}

// one persistent kernel per group size and layout: waves take work items
// from this class's queue until it is empty.
// Measured at K = 1000.  738M tokens in documents of 90: 85.5 ms on 32 lanes
// (103.7 with the spills that the opaque addresses took out, 118.5 with sorted
// topic lists kept token by token); of its eighth (92M tokens) 10.8 ms on 32
// lanes, 11.8 on 64, 12.5 on 16 and 12.9 on 8.  On 64 lanes a long document alone
// on its SIMD takes, by slots a lane, 0.23 us a token at 1, 0.34 at 3, 0.45 at 5,
// 0.60 at 8, 0.71 at 10, 0.81 at 12 and 1.11 at 16: the latency of one draw's
// chain, and about 0.05 us of instructions a slot.
// W: waves a SIMD that the registers leave room for (see fits_at_four_only).
template <int G, bool BIG, bool HOT, int W>
__global__ void __launch_bounds__(256, W) z_step_kernel(ZArgs a)
{
    extern __shared__ __align__(16) uint8_t z_lds[];
    // fp32(R_k) for the fp32 b-terms (the fp64 path reads R_k from global
    // memory)
    float *R = (float *)z_lds;
    for (int32_t k = threadIdx.x; k < a.m.K; k += blockDim.x) R[k] = (float)a.m.Rd[k];
    // the block's counters of the frequent words' increments
    uint32_t *hist = (uint32_t *)(z_lds + a.hot_off);
    const int32_t n_hist = HOT ? a.n_hot * a.m.K : 0;
    for (int32_t i = threadIdx.x; i < n_hist; i += blockDim.x) hist[i] = 0u;
    __syncthreads();
    const int wave = threadIdx.x >> 6;
    uint8_t *base = z_lds + a.r_bytes + wave * (64 / G) * a.lds.group_bytes;
    ZStat st;
    while (true) {
        int item = 0;
        if (__lane_id() == 0) item = atomicAdd(a.queue, 1);
        item = __builtin_amdgcn_readfirstlane(item);
        if (item >= a.n_items) break;
        // a private copy: a reference into global memory would be reloaded
        // after every store of the item (stores may alias it)
        const WorkItem w = a.items[item];
        z_step_item<G, BIG, HOT>(a, w, R, base, st, hist);
    }
    if (a.stats) {
        const unsigned long long j = wave_sum_u64(st.j), jb = wave_sum_u64(st.jb), na = wave_sum_u64(st.a),
                                 deg = wave_sum_u64(st.deg), fb = wave_sum_u64(st.fb);
        if (__lane_id() == 0) {
            if (j) atomicAdd(&a.stats[ST_SUM_J], j);
            if (na) atomicAdd(&a.stats[ST_SUM_A], na);
            if (deg) atomicAdd(&a.stats[ST_DEGENERATE], deg);
            if (jb) atomicAdd(&a.stats[ST_SUM_JB], jb);
            if (fb) atomicAdd(&a.stats[ST_FALLBACK], fb);
        }
    }
    if (HOT) {
        // every wave of the block is done: add the block's counters to n
        __syncthreads();
        const int32_t K = a.m.K;
        for (int32_t i = threadIdx.x; i < n_hist; i += blockDim.x) {
            const uint32_t c = hist[i];
            const int32_t h = i / K;
            if (c) atomicAdd(&a.m.n[(uint32_t)a.m.hot_word[h] * (uint32_t)K + (uint32_t)(i - h * K)], (int32_t)c);
        }
    }
}

// ---------------------------------------------------------------------------
// z-step, one document per lane (documents shorter than 128 tokens).  Lane l
// keeps its document's topics with a nonzero count as an ascending list of
// (topic, count) in LDS, entry j at j*64 + l so that the lanes' j-th entries
// are adjacent.  A token's b-terms are summed over the whole list in
// ascending topic order, one after the other in the lane (a listed topic
// the word's column lacks adds a zero term), so the running sums are those
// of the definition term by term.  The running sum after every block of 8
// entries stays in registers; the b-part walk re-reads one block.
// ---------------------------------------------------------------------------
constexpr int LANE_CAP = 127;                                      // list capacity
constexpr int LANE_BLK = 8;                                        // entries per gather batch
constexpr int LANE_NBLK = (LANE_CAP + LANE_BLK - 1) / LANE_BLK;    // 16

// first index j of the lane's list with topic >= key
__device__ __forceinline__ int32_t lane_lower_bound(const uint16_t *kl, int32_t L, int32_t key)
{
    int32_t lo = 0, hi = L;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if ((int32_t)kl[mid * 64] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// one block of the lane's list: b-terms of entries [j0, j0 + 8) (zero past L,
// and for a topic without a count, whatever its loaded phi)
template <bool VALUES>
__device__ __forceinline__ void lane_block_terms(const uint16_t *kl, const uint8_t *ml, int32_t L, int32_t j0,
                                                 const DevModel &M, uint32_t row, uint32_t fmt,
                                                 int32_t (&kk)[LANE_BLK], double (&bb)[LANE_BLK])
{
    uint32_t mm[LANE_BLK], xx[LANE_BLK];
#pragma unroll
    for (int u = 0; u < LANE_BLK; ++u) {
        const bool ok = j0 + u < L;
        const int32_t j = ok ? j0 + u : 0;
        const int32_t k = kl[j * 64];
        const uint32_t m = ml[j * 64];
        kk[u] = ok ? k : 0;
        mm[u] = ok ? m : 0u;
    }
    if constexpr (VALUES) {
#pragma unroll
        for (int u = 0; u < LANE_BLK; ++u) xx[u] = load_u32_at(M.phid, row + ((uint32_t)kk[u] << 2));
#pragma unroll
        for (int u = 0; u < LANE_BLK; ++u) bb[u] = (double)(mm[u] ? __uint_as_float(xx[u]) : 0.0f) * (double)mm[u];
        return;
    }
    double rr[LANE_BLK];
#pragma unroll
    for (int u = 0; u < LANE_BLK; ++u) {
        xx[u] = load_u32_at(M.gam, row + ((uint32_t)kk[u] << fmt)) & row_mask(fmt);
        rr[u] = M.Rd[kk[u]];
    }
    // phi_kv = fp32(x * R_k) == fp32(RN64(x / S_k)) for x < 0xFFFF and
    // S_k < 2^27; other draws divide
    float fk[LANE_BLK];
    bool far = false;
#pragma unroll
    for (int u = 0; u < LANE_BLK; ++u) {
        fk[u] = (float)((double)xx[u] * rr[u]);
        far |= xx[u] && (xx[u] >= 0xFFFFu || rr[u] <= 0x1p-27);
    }
    if (__builtin_amdgcn_ballot_w64(far)) {
#pragma unroll
        for (int u = 0; u < LANE_BLK; ++u)
            if (xx[u] && (xx[u] >= 0xFFFFu || rr[u] <= 0x1p-27)) fk[u] = (float)((double)xx[u] / (double)M.S[kk[u]]);
    }
#pragma unroll
    for (int u = 0; u < LANE_BLK; ++u) bb[u] = (double)fk[u] * (double)mm[u];
}

template <bool VALUES>
__global__ void __launch_bounds__(64) z_lane_kernel(ZArgs a)
{
    struct ZCount {
        unsigned long long J, A, degenerate;
    };
    extern __shared__ __align__(16) uint8_t l_lds[];
    const int lane = __lane_id();
    uint16_t *kl = (uint16_t *)l_lds + lane;                            // entry j at kl[j * 64]
    uint8_t *ml = l_lds + LANE_CAP * 64 * sizeof(uint16_t) + lane;      // entry j at ml[j * 64]
    const DevModel &M = a.m;
    const uint32_t t = *M.tptr;
    ZCount cnt = {0, 0, 0};
    while (true) {
        int item = 0;
        if (lane == 0) item = atomicAdd(a.queue, 1);
        item = __builtin_amdgcn_readlane(item, 0);
        if (item >= a.n_items) break;
        const WorkItem w = a.items[item];
        for (int32_t di = lane; di < w.count; di += 64) {
            const int32_t d = a.c.doc_order[w.first + di];
            const int64_t s = a.c.doc_off[d], e = a.c.doc_off[d + 1];
            // the document's counts as an ascending (topic, count) list
            int32_t L = 0;
            for (int64_t i = s; i < e; ++i) {
                const int32_t k = a.c.z[i];
                const int32_t pos = lane_lower_bound(kl, L, k);
                if (pos < L && kl[pos * 64] == k) {
                    ml[pos * 64] += 1;
                } else {
                    for (int32_t j = L - 1; j >= pos; --j) {
                        kl[(j + 1) * 64] = kl[j * 64];
                        ml[(j + 1) * 64] = ml[j * 64];
                    }
                    kl[pos * 64] = (uint16_t)k;
                    ml[pos * 64] = 1;
                    ++L;
                }
            }
            for (int64_t i = s; i < e; ++i) {
                const int32_t v = a.c.words[i];
                const int32_t kold = a.c.z[i];
                const int32_t cb = M.colptr[v];
                const int32_t Kv = M.colptr[v + 1] - cb;
                int32_t knew = kold;
                if (Kv == 0) {
                    // 0/0 conditional: the token keeps its topic
                    cnt.degenerate++;
                } else {
                    const r4 r = philox((uint32_t)i, (uint32_t)((uint64_t)i >> 32), t, TAG_Z, M.key0, M.key1);
                    const double sa = M.sigma_a[v];
                    const uint64_t al = M.calias[cb + scale32(r.y, (uint32_t)Kv)];
                    const int32_t ka = (r.z < (uint32_t)al) ? (int32_t)((al >> 32) & 0xFFFFu) : (int32_t)(al >> 48);
                    // m^{-i}
                    const int32_t po = lane_lower_bound(kl, L, kold);
                    const int32_t mo = ml[po * 64];
                    ml[po * 64] = (uint8_t)(mo - 1);
                    const int32_t Kd = L - (mo == 1 ? 1 : 0);
                    cnt.J += (unsigned long long)(Kd < Kv ? Kd : Kv);
                    const uint32_t fmt = VALUES ? ROW_32 : M.wrec[v].y >> 30;
                    const uint32_t row = VALUES ? (uint32_t)v * (uint32_t)M.K * 4u : draws_offset(M, fmt, v);
                    // sigma_b over the list, ascending, with the running sum after each block
                    double bs[LANE_NBLK];
                    double sb = 0.0;
                    int32_t last = -1;
    #pragma unroll
                    for (int blk = 0; blk < LANE_NBLK; ++blk) {
                        bs[blk] = sb;
                        if (!__builtin_amdgcn_ballot_w64(blk * LANE_BLK < L)) continue;
                        int32_t kk[LANE_BLK];
                        double bb[LANE_BLK];
                        lane_block_terms<VALUES>(kl, ml, L, blk * LANE_BLK, M, row, fmt, kk, bb);
    #pragma unroll
                        for (int u = 0; u < LANE_BLK; ++u) {
                            sb += bb[u];
                            if (bb[u] > 0.0) last = blk * LANE_BLK + u;
                        }
                        bs[blk] = sb;
                    }
                    const double x = unit24(r.x) * (sa + sb);
                    if (x < sa) {
                        knew = ka;
                        cnt.A++;
                    } else {
                        // b-part: the block whose running sum first passes y, then its entries
                        const double y = x - sa;
                        int32_t blk = -1;
                        double c0 = 0.0;
    #pragma unroll
                        for (int b = LANE_NBLK - 1; b >= 0; --b) {
                            if (bs[b] > y) {
                                blk = b;
                                c0 = b > 0 ? bs[b - 1] : 0.0;
                            }
                        }
                        knew = -1;
                        if (blk >= 0) {
                            int32_t kk[LANE_BLK];
                            double bb[LANE_BLK];
                            lane_block_terms<VALUES>(kl, ml, L, blk * LANE_BLK, M, row, fmt, kk, bb);
                            double c = c0;
    #pragma unroll
                            for (int u = 0; u < LANE_BLK; ++u) {
                                c += bb[u];
                                if (knew < 0 && bb[u] > 0.0 && c > y) knew = kk[u];
                            }
                        }
                        // no running sum passed y (rounding): the last positive term
                        if (knew < 0) knew = kl[last * 64];
                    }
                    // counts and list
                    if (knew == kold) {
                        ml[po * 64] = (uint8_t)mo;
                    } else {
                        if (mo == 1) {
                            for (int32_t j = po; j < L - 1; ++j) {
                                kl[j * 64] = kl[(j + 1) * 64];
                                ml[j * 64] = ml[(j + 1) * 64];
                            }
                            --L;
                        }
                        const int32_t pn = lane_lower_bound(kl, L, knew);
                        if (pn < L && kl[pn * 64] == knew) {
                            ml[pn * 64] += 1;
                        } else {
                            for (int32_t j = L - 1; j >= pn; --j) {
                                kl[(j + 1) * 64] = kl[j * 64];
                                ml[(j + 1) * 64] = ml[j * 64];
                            }
                            kl[pn * 64] = (uint16_t)knew;
                            ml[pn * 64] = 1;
                            ++L;
                        }
                    }
                    a.c.z[i] = (uint16_t)knew;
                }
                atomicAdd(&M.n[(uint32_t)v * (uint32_t)M.K + (uint32_t)knew], 1);
            }
            if (a.ll_doc) {
                // lgamma(A) - lgamma(N_d + A) + sum_k [lgamma(m_k + alpha) - lgamma(alpha)]
                double part = 0.0;
                for (int32_t j = 0; j < L; ++j) part += M.lg_alpha[ml[j * 64]];
                a.ll_doc[d] = part + M.lg_A[e - s];
            }
        }
    }
    if (a.stats) {
        if (cnt.J) {
            atomicAdd(&a.stats[ST_SUM_J], (unsigned long long)cnt.J);
            atomicAdd(&a.stats[ST_SUM_JB], (unsigned long long)cnt.J);
        }
        if (cnt.A) atomicAdd(&a.stats[ST_SUM_A], (unsigned long long)cnt.A);
        if (cnt.degenerate) atomicAdd(&a.stats[ST_DEGENERATE], (unsigned long long)cnt.degenerate);
    }
}

static int ilog2(int x)
{
    int r = 0;
    while ((1 << r) < x) ++r;
    return r;
}

static int topics_per_lane_log2(int K, int G)
{
    int c = ilog2((K + G - 1) / G);
    return c;
}

// what a z-step starts from: no counts, empty queues, one more z-step counted
__global__ void __launch_bounds__(256) z_prepare_kernel(int32_t *n, int64_t cells, int32_t *queues,
                                                        unsigned long long *stats)
{
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t quads = cells >> 2;   // (the table is 256-byte aligned)
    for (int64_t i = i0; i < quads; i += (int64_t)gridDim.x * blockDim.x) ((int4 *)n)[i] = make_int4(0, 0, 0, 0);
    if (i0 < (cells & 3)) n[4 * quads + i0] = 0;
    if (blockIdx.x == 0) {
        if (threadIdx.x < Z_QUEUES) queues[threadIdx.x] = 0;
        if (threadIdx.x == 0 && stats) stats[ST_TOKENS] += 1ull;
    }
}

hipError_t launch_z_prepare(const DevModel &m, int32_t *queues, unsigned long long *stats, hipStream_t s)
{
    const int64_t cells = m.n ? (int64_t)m.V * m.K : 0;
    z_prepare_kernel<<<grid_for(cells / 4, 256, 16384), 256, 0, s>>>(m.n, cells, queues, stats);
    return hipGetLastError();
}

// Registers of the token kernels.  At 4 waves a SIMD (128 registers) the
// longest lists' kernels on 64 lanes spill 70 to 100 of them, at 3 (168) few or
// none, and draw faster: z-step of 20,000 documents of 700 tokens at K = 1000
// 2.67 and 2.37 ms.  But where the work is one wave each (a document, a
// request) and fits the chip at once at 4 and not at 3, the second round costs
// more: 4,000 documents of 3,000 tokens 3.86 and 4.31 ms, fold-in of 4,096
// requests of 300 tokens at K = 100 2.97 and 3.39 ms.
static bool fits_at_four_only(int64_t blocks, int32_t n_cu) { return blocks > 3 * (int64_t)n_cu && blocks <= 4 * (int64_t)n_cu; }

hipError_t launch_z_class(const DevCorpus &c, const DevModel &m, int32_t group, int32_t longest,
                          const WorkItem *items, int32_t n_items, int32_t n_cu, int32_t *queue, unsigned long long *stats,
                          double *ll_doc, hipStream_t s)
{
    if (n_items == 0) return hipSuccess;
    if (!z_group_fits(group, m.K, longest)) return hipErrorInvalidValue;
    ZArgs a;
    a.m = m;
    a.c = c;
    a.items = items;
    a.n_items = n_items;
    a.queue = queue;
    a.stats = stats;
    a.ll_doc = m.lg_alpha ? ll_doc : nullptr;
    a.lds = slot_lds(group, m.K, longest);
    a.r_bytes = (m.K * 4 + 15) / 16 * 16;
    size_t lds = (size_t)a.r_bytes + 4 * (size_t)(group == 1 ? 0 : 64 / group) * a.lds.group_bytes;
    a.n_hot = 0;
    a.hot_off = (int32_t)lds;
    auto launch = [&](auto kernel, auto kernel_hot) -> hipError_t {
        // persistent: exactly the blocks the device holds at once, and no
        // more waves than work items (a wave takes one item at a time)
        int per_cu = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, lds);
        if (e != hipSuccess) return e;
        bool hot = false;
        if (m.n_hot > 0) {
            // the frequent words' counters in LDS, unless they cost blocks
            const size_t with = lds + (size_t)m.n_hot * m.K * 4;
            int per_cu_hot = 0;
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_hot, kernel_hot, 256, with);
            if (e != hipSuccess) return e;
            if (per_cu_hot == per_cu) {
                a.n_hot = m.n_hot;
                lds = with;
                hot = true;
            }
        }
        if (per_cu <= 0) return hipErrorInvalidConfiguration;  // the block's LDS exceeds the CU's
        int64_t blocks = (int64_t)per_cu * (n_cu > 0 ? n_cu : 1);
        const int64_t need = ((int64_t)n_items + 3) / 4;
        if (blocks > need) blocks = need;
        if (hot) kernel_hot<<<(unsigned)blocks, 256, lds, s>>>(a);
        else kernel<<<(unsigned)blocks, 256, lds, s>>>(a);
        return hipGetLastError();
    };
    if (group == 1) {
        // one document per lane: 64-thread blocks, the lanes' topic lists
        const size_t llds = (size_t)LANE_CAP * 64 * 3;
        auto kernel = m.values ? z_lane_kernel<true> : z_lane_kernel<false>;
        int per_cu = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 64, llds);
        if (e != hipSuccess) return e;
        if (per_cu <= 0) return hipErrorInvalidConfiguration;
        int64_t blocks = (int64_t)per_cu * (n_cu > 0 ? n_cu : 1);
        if (blocks > n_items) blocks = n_items;
        kernel<<<(unsigned)blocks, 64, llds, s>>>(a);
        return hipGetLastError();
    }
    const bool big = a.lds.slots > SLOTS_FEW;
    if (group == 64) {
        if (!big) return launch(z_step_kernel<64, false, false, 3>, z_step_kernel<64, false, true, 3>);
        // (more than 384 topics: no frequent words' counters)
        if (fits_at_four_only(((int64_t)n_items + 3) / 4, n_cu))
            return launch(z_step_kernel<64, true, false, 4>, z_step_kernel<64, true, false, 4>);
        return launch(z_step_kernel<64, true, false, 3>, z_step_kernel<64, true, false, 3>);
    }
#define PULDA_Z(G_)                                                                                      \
    (big ? launch(z_step_kernel<G_, true, false, 3>, z_step_kernel<G_, true, true, 3>)                   \
         : launch(z_step_kernel<G_, false, false, 4>, z_step_kernel<G_, false, true, 4>))
    if (group == 32) return PULDA_Z(32);
    if (group == 16) return PULDA_Z(16);
    return PULDA_Z(8);
#undef PULDA_Z
}

// ---------------------------------------------------------------------------
// Collapsed log joint (Section 4 reports it per iteration):
//   words: K lgamma(V beta) - sum_k lgamma(n_k + V beta)
//          + sum_{k,v: n_kv > 0} [lgamma(n_kv + beta) - lgamma(beta)]
//   docs:  sum_d [lgamma(A) - lgamma(N_d + A)
//          + sum_{k: m_dk > 0} (lgamma(m_dk + alpha_k) - lgamma(alpha_k))]
// Two launches.  The first reads the counts once: a block adds its words'
// counts by topic in LDS beside the cells' terms, and writes one row of
// partial sums; its other blocks take the documents.  The second adds the rows up by topic, and
// its last block to finish adds everything else.  Partial sums are added in a
// fixed order, so the value is the same on every run.
// Measured at V = 28,000, K = 1000 and 200,000 documents of 90 tokens: 117 +
// 17 us, from 330 us when the counts were read twice (50 + 53 us) and every
// document cleared and read a table of K counts (215 us).  The words alone take
// 55 us (112 MB of counts: the table lookups and LDS adds of 28M cells), the
// documents alone 75 us.  Bound by latency at two waves a SIMD (199 registers, the
// rare cells' lgamma and log inlined): the VALU is busy 39% of the cycles, a wave
// waits in 53% of its own.
// ---------------------------------------------------------------------------
constexpr int32_t LL_DOCS = 256;   // documents' terms per block, at least

__device__ __forceinline__ double block_sum_f64(double x, double *red)
{
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int wv = 0; wv < (int)(blockDim.x >> 6); ++wv) t += red[wv];
    return t;
}

struct LLArgs {
    const int32_t *n;
    int32_t V, K;
    int32_t words;              // words per block of the words' part
    int32_t nw, nd;             // blocks of the words' part, of the documents'
    double beta, lgb;
    const double *lg_beta, *beta_v;
    unsigned long long *part_nk;   // [nw * K]
    double *part;                  // [nw + nd], then [ceil(K / 16)] of the second launch
    unsigned long long *nk;        // [K]
    DevCorpus c;
    const double *ll_doc;          // the documents' terms, or null: counted from z
    const double *alpha, *lg_alpha, *lg_A;   // (lg_alpha: symmetric alpha only)
    int32_t symmetric;
    int32_t longest;               // tokens past which a document is counted by a block
    uint32_t *done;                // blocks of the second launch that have finished
    double Vbeta, *out, *hist;
    const uint32_t *hist_idx;
    uint32_t *advance_t, *advance_hist;   // sweep number and history index, moved on when set
};

// The words' part: a block's cells in one run, U a thread in flight.  A cell's term is lgamma(n + beta) - lgamma(beta), by table for the symmetric
// beta (an entry of zero for n = 0, so that every lane reads without a
// branch); with per-word priors log(beta (beta + 1) .. (beta + n - 1)) for
// small counts.  Counts are added to their topic in LDS.
__device__ __forceinline__ double ll_words(const LLArgs &a, unsigned long long *sum)
{
    const int tid = threadIdx.x;
    const int32_t K = a.K;
    const int32_t v0 = blockIdx.x * a.words;
    const int64_t c0 = (int64_t)v0 * K;
    const int64_t c1 = (int64_t)(v0 + a.words < a.V ? v0 + a.words : a.V) * K;
    for (int32_t k = tid; k < K; k += 256) sum[k] = 0;
    __syncthreads();
    double acc = 0.0;
    constexpr int U = 16;
    const int32_t dv = 256 / K, dk = 256 - dv * K;   // a turn's step in words and topics
    int32_t v = v0 + tid / K, k = tid % K;
    const int32_t *n0 = a.n + c0 + tid;
    const int32_t cells = (int32_t)(c1 - c0);
    for (int32_t cb = 0; cb < cells; cb += 256 * U) {
        int32_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = cb + 256 * u + tid < cells ? n0[cb + 256 * u] : 0;
        if (!a.beta_v) {
            double t[U];
            bool far = false;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = (uint32_t)x[u] < (uint32_t)LG_TABLE;
                t[u] = a.lg_beta[in ? x[u] : 0];
                far |= !in;
            }
#pragma unroll
            for (int u = 0; u < U; u += 4) acc += (t[u] + t[u + 1]) + (t[u + 2] + t[u + 3]);
            if (far) {
#pragma unroll 1
                for (int u = 0; u < U; ++u) {
                    const int32_t c = cb + 256 * u + tid < cells ? n0[cb + 256 * u] : 0;
                    if (c >= LG_TABLE) acc += lgamma((double)c + a.beta) - a.lgb;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            atomicAdd(&sum[k], (unsigned long long)(uint32_t)x[u]);
            if (a.beta_v && x[u] > 0) {
                const double b = a.beta_v[v];
                if (x[u] <= 8) {
                    double p = b;
                    for (int q = 1; q < x[u]; ++q) p *= b + (double)q;
                    acc += log(p);
                } else {
                    acc += lgamma((double)x[u] + b) - lgamma(b);
                }
            }
            v += dv;
            k += dk;
            if (k >= K) {
                k -= K;
                ++v;
            }
        }
    }
    __syncthreads();
    unsigned long long *row = a.part_nk + (int64_t)blockIdx.x * K;
    for (int32_t q = tid; q < K; q += 256) row[q] = sum[q];
    return acc;
}

// Documents counted from z, a wave to a document: sum over topics of
// lgamma(m + alpha_k) - lgamma(alpha_k) = sum over the tokens of
// log(alpha_k + j), j the tokens of the topic counted before (LDS handles a
// wave's adds to one address in lane order).  So no table of K counts is
// cleared or read per document: the tokens clear what they counted.  The
// offsets of 64 documents and the next document's first tokens are in flight
// while one is counted.
// A document much longer than a wave's share would be a chain behind all
// others: the wave sets it aside, and the block then counts it together, with
// the terms of its topics by table (a sum over tokens would depend on which of
// the waves' tokens came first).  4,000 documents of 20 tokens and one of
// 65,535: 360 us a log joint in a wave, 55 so.
constexpr int32_t LL_LONG = 1024;  // fewest tokens of such a document
constexpr int32_t LL_ASIDE = 32;   // of them per wave; the others stay in the wave
constexpr int32_t LL_LOGS = 256;   // log(alpha + j) in LDS (symmetric alpha), and a zero
constexpr int32_t LL_IDLE = 64;    // a count for each lane without a token

inline size_t ll_docs_lds(int32_t K)
{
    return (LL_LOGS + 1) * sizeof(double) + 4 * ((size_t)(K + 1) / 2 + LL_IDLE) * sizeof(uint32_t);
}

struct LLAside {
    int32_t n[4], doc[4][LL_ASIDE];
};

// LONG: there are documents to set aside (a kernel of its own: the code for
// them takes 3% more time where there are none)
template <bool SYM, bool LONG>
__device__ __forceinline__ double ll_docs(const LLArgs &a, uint8_t *lds, LLAside *aside)
{
    const int lane = __lane_id(), wv = threadIdx.x >> 6;
    double *logs = (double *)lds;
    const int32_t words = (a.K + 1) / 2 + LL_IDLE;
    uint32_t *cnt = (uint32_t *)(lds + (LL_LOGS + 1) * sizeof(double)) + wv * words;
    const int32_t idle = 2 * (words - LL_IDLE + lane);   // the "topic" of no token
    for (int32_t i = lane; i < words; i += 64) cnt[i] = 0;
    if (SYM) {
        logs[threadIdx.x] = log(a.alpha[0] + (double)threadIdx.x);
        if (threadIdx.x == 0) logs[LL_LOGS] = 0.0;
    }
    __syncthreads();
    const int64_t waves = (int64_t)a.nd * 4;
    const int64_t per = (a.c.D + waves - 1) / waves;
    const int64_t d0 = ((int64_t)(blockIdx.x - a.nw) * 4 + wv) * per;
    const int64_t d1 = d0 + per < a.c.D ? d0 + per : a.c.D;
    constexpr int C = 4;   // 64-token chunks at a time
    const uint16_t *zl = a.c.z + lane;
    double acc = 0.0;
    int32_t n_aside = 0;
    // C chunks of a document's tokens from token p
    auto load = [&](int64_t s, int32_t p, int32_t n, int32_t (&k)[C]) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            k[c] = idle;
            if (p + 64 * c < n && p + 64 * c + lane < n) k[c] = zl[s + p + 64 * c];
        }
    };
    auto count = [&](int32_t p, int32_t n, const int32_t (&k)[C]) {
        uint32_t was[C];
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (p + 64 * c < n) was[c] = atomicAdd(&cnt[k[c] >> 1], 1u << (16 * (k[c] & 1)));
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (p + 64 * c >= n) continue;
            const int32_t j = (int32_t)__builtin_amdgcn_ubfe(was[c], 16 * (k[c] & 1), 16);
            const bool on = k[c] < idle - 2 * lane;
            if (SYM) {
                acc += logs[on && j < LL_LOGS ? j : LL_LOGS];
                if (__builtin_amdgcn_ballot_w64(on && j >= LL_LOGS)) acc += on && j >= LL_LOGS ? log(a.alpha[0] + (double)j) : 0.0;
            } else if (on) {
                acc += log(a.alpha[k[c]] + (double)j);
            }
        }
    };
    auto clear = [&](int32_t p, int32_t n, const int32_t (&k)[C]) {
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (p + 64 * c < n) cnt[k[c] >> 1] = 0;
    };
    for (int64_t db = d0; db < d1; db += 64) {
        const int nb = (int)(d1 - db < 64 ? d1 - db : 64);
        int64_t off = 0;
        int32_t len = 0;
        if (lane < nb) {
            off = a.c.doc_off[db + lane];
            len = (int32_t)(a.c.doc_off[db + lane + 1] - off);
            acc += a.lg_A[len];
        }
        // (set aside: empty for the wave)
        const uint64_t big = LONG ? __builtin_amdgcn_ballot_w64(len > a.longest) : 0;
        if (big != 0) {
            const int32_t at = n_aside + __builtin_popcountll(big & ((1ull << lane) - 1ull));
            if (len > a.longest && at < LL_ASIDE) {
                aside->doc[wv][at] = (int32_t)(db + lane);
                len = 0;
            }
            n_aside += __builtin_popcountll(big);
            n_aside = n_aside < LL_ASIDE ? n_aside : LL_ASIDE;
        }
        int64_t s = 0;
        int32_t n = 0, z[C];
        auto next = [&](int i) {
            s = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)off, i) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(off >> 32), i) << 32);
            n = __builtin_amdgcn_readlane(len, i);
            load(s, 0, n, z);
        };
        next(0);
        for (int i = 0; i < nb; ++i) {
            const int64_t sd = s;
            const int32_t nd = n;
            int32_t k[C];
#pragma unroll
            for (int c = 0; c < C; ++c) k[c] = z[c];
            if (i + 1 < nb) next(i + 1);
            count(0, nd, k);
            if (nd > 64 * C) {
                // a long document: the next chunks in flight while these are
                // counted, and the table cleared whole
                int32_t a1[C], a2[C];
                load(sd, 64 * C, nd, a1);
                for (int32_t p = 64 * C; p < nd; p += 64 * C) {
                    load(sd, p + 64 * C, nd, a2);
                    count(p, nd, a1);
#pragma unroll
                    for (int c = 0; c < C; ++c) a1[c] = a2[c];
                }
                lds_order();
                for (int32_t w = lane; w < words; w += 64) cnt[w] = 0;
            }
            lds_order();
            clear(0, nd, k);
            lds_order();
        }
    }
    if constexpr (!LONG) return acc;
    // the documents set aside, the block's tables as one of K counts
    if (lane == 0) aside->n[wv] = n_aside;
    uint32_t *all = (uint32_t *)(lds + (LL_LOGS + 1) * sizeof(double));
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        for (int32_t j = 0; j < aside->n[w]; ++j) {
            const int32_t d = aside->doc[w][j];
            const int64_t s = a.c.doc_off[d];
            const int32_t n = (int32_t)(a.c.doc_off[d + 1] - s);
            constexpr int U = 16;
            for (int32_t p = threadIdx.x; p < n; p += 256 * U) {
                int32_t k[U];
#pragma unroll
                for (int u = 0; u < U; ++u) k[u] = p + 256 * u < n ? a.c.z[s + p + 256 * u] : -1;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (k[u] >= 0) atomicAdd(&all[k[u]], 1u);
            }
            __syncthreads();
            for (int32_t k = threadIdx.x; k < a.K; k += 256) {
                const uint32_t c = all[k];
                all[k] = 0;
                if (SYM) acc += c ? a.lg_alpha[c] : 0.0;
                else if (c) acc += lgamma((double)c + a.alpha[k]) - lgamma(a.alpha[k]);
            }
            __syncthreads();
        }
    }
    return acc;
}

// COUNT: documents counted from z; else their terms as the z-step left them
template <bool COUNT, bool LONG>
__global__ void __launch_bounds__(256) ll_terms_kernel(LLArgs a)
{
    extern __shared__ __align__(16) uint8_t ll_lds[];
    __shared__ double red[4];
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.done = 0;
    double acc = 0.0;
    if ((int)blockIdx.x < a.nw) {
        unsigned long long *sum = (unsigned long long *)ll_lds;
        acc = ll_words(a, sum);
    } else if constexpr (COUNT) {
        LLAside *aside = nullptr;
        if constexpr (LONG) {
            __shared__ LLAside lists;
            aside = &lists;
        }
        acc = a.symmetric ? ll_docs<true, LONG>(a, ll_lds, aside) : ll_docs<false, LONG>(a, ll_lds, aside);
    } else {
        const int64_t per = (a.c.D + a.nd - 1) / a.nd;
        const int64_t d0 = (int64_t)(blockIdx.x - a.nw) * per, d1 = d0 + per < a.c.D ? d0 + per : a.c.D;
        for (int64_t d = d0 + threadIdx.x; d < d1; d += 256) acc += a.ll_doc[d];
    }
    const double t = block_sum_f64(acc, red);
    if (threadIdx.x == 0) a.part[blockIdx.x] = t;
}

// 16 topics to a block, 64 threads to a topic
__global__ void __launch_bounds__(1024) ll_final_kernel(LLArgs a)
{
    __shared__ unsigned long long sums[256];
    __shared__ double red[16];
    __shared__ int last;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int32_t k = blockIdx.x * 16 + (tid & 15);
    unsigned long long s = 0;
    if (k < a.K)
        for (int32_t r = tid >> 4; r < a.nw; r += 64) s += a.part_nk[(int64_t)r * a.K + k];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (lane < 16) sums[w * 16 + lane] = s;
    __syncthreads();
    double acc = 0.0;
    if (tid < 16 && k < a.K) {
        s = 0;
        for (int j = 0; j < 16; ++j) s += sums[j * 16 + tid];
        a.nk[k] = s;
        acc = -lgamma((double)s + a.Vbeta);
    }
    const int32_t np = a.nw + a.nd;
    double t = block_sum_f64(acc, red);
    if (tid == 0) {
        a.part[np + blockIdx.x] = t;
        __threadfence();
        last = atomicAdd(a.done, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    acc = 0.0;
    for (int32_t i = tid; i < np + (int32_t)gridDim.x; i += 1024)
        acc += __hip_atomic_load(&a.part[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    t = block_sum_f64(acc, red);
    if (tid == 0) {
        const double ll = (double)a.K * lgamma(a.Vbeta) + t;
        *a.out = ll;
        if (a.hist) a.hist[*a.hist_idx] = ll;
        if (a.advance_t) {
            *a.advance_t += 1u;
            *a.advance_hist += 1u;
        }
    }
}

__global__ void set_sweep_kernel(uint32_t *tptr, uint32_t t, uint32_t *hist_idx)
{
    if (threadIdx.x == 0) {
        *tptr = t;
        *hist_idx = 0u;
    }
}

hipError_t launch_set_sweep(uint32_t *tptr, uint32_t t, uint32_t *hist_idx, hipStream_t s)
{
    set_sweep_kernel<<<1, 64, 0, s>>>(tptr, t, hist_idx);
    return hipGetLastError();
}

hipError_t launch_loglik(const DevCorpus &c, const DevModel &m, const LLSpace &space, const double *ll_doc, double *out,
                         double *hist, uint32_t *hist_idx, uint32_t *advance_t, hipStream_t s)
{
    LLArgs a;
    a.n = m.n;
    a.V = m.V;
    a.K = m.K;
    // at least a turn of the block's cells, and of K sums
    const int32_t share = (m.V + space.max_words - 1) / space.max_words, least = 4096 / m.K + 4;
    a.words = share > least ? share : least;
    a.nw = (m.V + a.words - 1) / a.words;
    // a block for 16 documents; for 4,096 tokens while that is more and there
    // are few (long documents on an idle chip)
    int64_t docs = (c.D + LL_DOCS - 1) / LL_DOCS;
    if (!ll_doc) {
        const int64_t few = c.N / 4096 < 512 ? c.N / 4096 : 512;
        docs = (c.D + 15) / 16 > few ? (c.D + 15) / 16 : few;
    }
    a.nd = (int32_t)(docs < 1 ? 1 : (docs < space.max_docs ? docs : space.max_docs));
    const int64_t share_tokens = c.N / (4 * (int64_t)a.nd);   // of a wave
    a.longest = (int32_t)(share_tokens < LL_LONG ? LL_LONG : (share_tokens < 65536 ? share_tokens : 65536));
    a.beta = m.beta;
    a.lgb = lgamma(m.beta);
    a.lg_beta = m.lg_beta;
    a.beta_v = m.beta_v;
    a.part_nk = space.part_nk;
    a.part = space.part;
    a.nk = m.nk;
    a.c = c;
    a.ll_doc = ll_doc;
    a.alpha = m.alpha;
    a.lg_alpha = m.lg_alpha;
    a.lg_A = m.lg_A;
    a.symmetric = m.lg_alpha != nullptr;
    a.done = space.done;
    a.Vbeta = m.beta_sum;
    a.out = out;
    a.hist = hist;
    a.hist_idx = hist_idx;
    a.advance_t = advance_t;
    a.advance_hist = hist_idx;
    const size_t sums = (size_t)m.K * 8;
    if (ll_doc) {
        ll_terms_kernel<false, false><<<a.nw + a.nd, 256, sums, s>>>(a);
    } else {
        const size_t tables = ll_docs_lds(m.K), lds = sums > tables ? sums : tables;
        if (c.longest > a.longest) ll_terms_kernel<true, true><<<a.nw + a.nd, 256, lds, s>>>(a);
        else ll_terms_kernel<true, false><<<a.nw + a.nd, 256, lds, s>>>(a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    ll_final_kernel<<<(m.K + 15) / 16, 1024, 0, s>>>(a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Phi export / import (parity tests; serving models built elsewhere)
// ---------------------------------------------------------------------------
__global__ void export_phi_kernel(DevModel m, int64_t *colptr64, uint16_t *topic, int32_t *gam_e, float *phi_e,
                                  uint32_t *thr, uint16_t *alias_topic)
{
    const int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= m.V) return;
    const int lane = __lane_id();
    const int32_t a = m.colptr[v], b = m.colptr[v + 1];
    const uint32_t fmt = m.wrec[v].y >> 30;
    if (lane == 0) {
        colptr64[v] = a;
        if (v == m.V - 1) colptr64[m.V] = b;
    }
    for (int32_t e = a + lane; e < b; e += 64) {
        const int32_t k = m.ctopic[e];
        topic[e] = (uint16_t)k;
        phi_e[e] = m.cphi[e];
        gam_e[e] = m.phi_method == 1 ? 0 : (int32_t)row_draw(m, fmt, v, k);
        const uint64_t al = m.calias[e];
        thr[e] = (uint32_t)al;
        alias_topic[e] = (uint16_t)(al >> 48);
    }
}

hipError_t launch_export_phi(const DevModel &m, int64_t *colptr64, uint16_t *topic, int32_t *gam_e, float *phi_e,
                             uint32_t *thr, uint16_t *alias_topic, hipStream_t s)
{
    export_phi_kernel<<<(m.V + 3) / 4, 256, 0, s>>>(m, colptr64, topic, gam_e, phi_e, thr, alias_topic);
    return hipGetLastError();
}

__global__ void import_phi_kernel(DevModel m, const int64_t *colptr64, const uint16_t *topic, const float *phi_e,
                                  const uint32_t *thr, const uint16_t *alias_topic)
{
    const int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= m.V) return;
    const int lane = __lane_id();
    const int64_t a = colptr64[v], b = colptr64[v + 1];
    if (lane == 0) {
        m.colptr[v] = (int32_t)a;
        if (v == m.V - 1) m.colptr[m.V] = (int32_t)b;
    }
    float *pcol = m.phid + (int64_t)v * m.K;
    for (int32_t k = lane; k < m.K; k += 64) pcol[k] = 0.0f;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    // values without draws behind them: every nonzero cell is read from phid
    float fmax = 0.0f;
    for (int64_t e = a + lane; e < b; e += 64) {
        const int32_t k = topic[e];
        fmax = phi_e[e] > fmax ? phi_e[e] : fmax;
        m.ctopic[e] = (uint16_t)k;
        m.cphi[e] = phi_e[e];
        pcol[k] = phi_e[e];
        m.calias[e] = (uint64_t)thr[e] | ((uint64_t)k << 32) | ((uint64_t)alias_topic[e] << 48);
    }
    for (int o = 32; o > 0; o >>= 1) {
        const float y = __shfl_xor(fmax, o, 64);
        fmax = y > fmax ? y : fmax;
    }
    if (lane == 0) m.phimax[v] = __float_as_uint(fmax);
}

hipError_t launch_import_phi(const DevModel &m, const int64_t *colptr64, const uint16_t *topic, const float *phi_e,
                             const uint32_t *thr, const uint16_t *alias_topic, hipStream_t s)
{
    import_phi_kernel<<<(m.V + 3) / 4, 256, 0, s>>>(m, colptr64, topic, phi_e, thr, alias_topic);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// counts export: n as CSC by word (ascending topic), m as CSR by document
// ---------------------------------------------------------------------------
__global__ void n_colcount_kernel(const int32_t *n, int32_t V, int32_t K, int64_t *cnt)
{
    const int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= V) return;
    const int lane = __lane_id();
    int32_t c = 0;
    for (int32_t k = lane; k < K; k += 64) c += n[(int64_t)v * K + k] > 0;
    c = group_scan_incl_i32<64>(c);
    if (lane == 63) cnt[v] = c;
}

__global__ void n_fill_kernel(const int32_t *n, int32_t V, int32_t K, const int64_t *colptr, uint16_t *topic,
                              int32_t *cnt)
{
    const int32_t v = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (v >= V) return;
    const int lane = __lane_id();
    int64_t run = colptr[v];
    for (int32_t k0 = 0; k0 < K; k0 += 64) {
        const int32_t k = k0 + lane;
        const int32_t x = k < K ? n[(int64_t)v * K + k] : 0;
        const uint64_t bal = __builtin_amdgcn_ballot_w64(x > 0);
        if (x > 0) {
            const int64_t e = run + __builtin_popcountll(bal & ((1ull << lane) - 1ull));
            topic[e] = (uint16_t)k;
            cnt[e] = x;
        }
        run += __builtin_popcountll(bal);
    }
}

hipError_t launch_counts_csc(const DevModel &m, const int64_t *colptr64, uint16_t *topic, int32_t *cnt,
                             int32_t *unused, hipStream_t s)
{
    (void)unused;
    n_fill_kernel<<<(m.V + 3) / 4, 256, 0, s>>>(m.n, m.V, m.K, colptr64, topic, cnt);
    return hipGetLastError();
}

// pass 0: per-column / per-document nonzero counts (int64) into rowcnt
// pass 1: fill CSR m with rowptr = rowcnt (already scanned)
__global__ void m_rows_kernel(DevCorpus c, int32_t K, int32_t log2c, int64_t *rowcnt_or_ptr, uint16_t *topic,
                              int32_t *cnt, int pass)
{
    extern __shared__ uint16_t m_lds[];
    const int lane = __lane_id();
    const int wv = threadIdx.x >> 6;
    const int32_t C = 1 << log2c;
    uint16_t *mt = m_lds + wv * (64 * C);
    const int64_t d = blockIdx.x * 4 + wv;
    if (d >= c.D) return;
    const int64_t s = c.doc_off[d], e = c.doc_off[d + 1];
    for (int32_t i = lane; i < 64 * C; i += 64) mt[i] = 0;
    __builtin_amdgcn_wave_barrier();
    for (int64_t i = s + lane; i < e; i += 64) {
        const int32_t k = c.z[i];
        const int32_t slot = (k & (C - 1)) * 64 + (k >> log2c);
        atomicAdd((uint32_t *)(mt + (slot & ~1)), (slot & 1) ? 65536u : 1u);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int32_t mine = 0;
    for (int32_t b = 0; b < C; ++b) mine += mt[b * 64 + lane] > 0;
    const int32_t incl = group_scan_incl_i32<64>(mine);
    if (pass == 0) {
        if (lane == 63) rowcnt_or_ptr[d] = incl;
        return;
    }
    int64_t o = rowcnt_or_ptr[d] + incl - mine;
    for (int32_t b = 0; b < C; ++b) {
        const int32_t x = mt[b * 64 + lane];
        if (x > 0) {
            topic[o] = (uint16_t)(lane * C + b);
            cnt[o] = x;
            ++o;
        }
    }
}

hipError_t launch_counts_m(const DevCorpus &c, int32_t K, int64_t *rowcnt_or_ptr, uint16_t *topic, int32_t *cnt,
                           int pass, hipStream_t s)
{
    if (c.D == 0) return hipSuccess;
    const int log2c = topics_per_lane_log2(K, 64);
    m_rows_kernel<<<(unsigned)((c.D + 3) / 4), 256, 4 * 64 * (1 << log2c) * sizeof(uint16_t), s>>>(
        c, K, log2c, rowcnt_or_ptr, topic, cnt, pass);
    return hipGetLastError();
}

hipError_t launch_n_colcount(const DevModel &m, int64_t *cnt, hipStream_t s)
{
    n_colcount_kernel<<<(m.V + 3) / 4, 256, 0, s>>>(m.n, m.V, m.K, cnt);
    return hipGetLastError();
}

hipError_t launch_scan_i64(const int64_t *in, int64_t *out_excl, int64_t n, long long *scratch, hipStream_t s)
{
    return scan_excl<int64_t, int64_t>(in, out_excl, n, scratch, scratch + (n + SCAN_BLOCK - 1) / SCAN_BLOCK, s);
}

// ---------------------------------------------------------------------------
// Fold-in (Phi fixed, no count rebuild): each group owns one request slot.
// On its first step a slot drops tokens whose word is out of range or has an
// empty Phi column, and draws initial topics.  Every step then runs up to
// `budget` token draws, resuming where the previous step stopped (sweep and
// token within it, kept on the device), with counters (p, request, sweep):
// the draws do not depend on how a request's work is cut into steps.  The
// topic counts are accumulated after each sweep past the burn-in, and the
// step that ends the last sweep writes theta and the log-likelihood of the
// final state.
// ---------------------------------------------------------------------------
template <int G, bool SYM>
__device__ __forceinline__ void foldin_slot(const DevModel &M, const DevFoldin &F, int32_t sid, const float *Rf,
                                            uint8_t *base, const SlotLds &A)
{
    SlotDoc S = slot_doc(base, A);
    const int lane = __lane_id();
    const int g = lane & (G - 1);
    const int32_t K = M.K;
    const FoldSlot sl = F.slots[sid];
    int32_t *wds = F.words + sl.arena_off;
    int32_t *pos = F.pos + sl.arena_off;
    uint16_t *zz = F.z + sl.arena_off;
    uint32_t *acc = F.acc + (int64_t)sid * K;
    int32_t kept = 0, done = 0, next = 0;
    if (sl.fresh) {
        // drop tokens, compact the kept positions, draw initial topics
        int32_t run = 0;
        for (int32_t p0 = 0; p0 < sl.len; p0 += G) {
            const int32_t p = p0 + g;
            int32_t v = -1;
            bool keep = false;
            if (p < sl.len) {
                v = wds[p];
                keep = v >= 0 && v < M.V && M.colptr[v + 1] > M.colptr[v];
            }
            const uint64_t bal = group_ballot<G>(keep);
            if (keep) {
                // (the kept words move up in place: q <= p, and this block's
                // words have been read)
                const int32_t q = run + __builtin_popcountll(bal & ((1ull << g) - 1ull));
                pos[q] = p;
                wds[q] = v;
                const r4 r = philox((uint32_t)p, sl.req, 0u, TAG_FOLDIN_INIT, F.key0, F.key1);
                zz[q] = (uint16_t)scale32(r.x, (uint32_t)K);
            }
            run += __builtin_popcountll(bal);
        }
        kept = run;
        for (int32_t k = g; k < K; k += G) acc[k] = 0;
        if (g == 0) {
            F.kept[2 * sid] = kept;
            F.kept[2 * sid + 1] = sl.len - kept;
            F.fin[sid] = 0;
        }
        __threadfence();
    } else {
        kept = F.kept[2 * sid];
        done = F.prog[2 * sid];
        next = F.prog[2 * sid + 1];
        // finished in an earlier step (a step launched before the host
        // collected it): its results stay as they are
        if (done >= F.sweeps) return;
    }
    slots_load<G, false>(S, A, zz, 0, kept, g);
    ZStat st;
    int32_t budget = sl.budget;
    while (budget > 0 && done < F.sweeps) {
        const int32_t s = done + 1;
        const int32_t t1 = kept - next < budget ? kept : next + budget;
        for (int32_t q0 = next; q0 < t1; q0 += G) {
            const int32_t q = q0 + g;
            const bool valid = q < t1;
            int32_t zo = 0;
            LaneTok x = no_token();
            if (valid) {
                const int32_t p = pos[q];
                zo = zz[q];
                const r4 r = philox((uint32_t)p, sl.req, (uint32_t)s, TAG_FOLDIN_Z, F.key0, F.key1);
                x = stage_token(M, wds[q], zo, r, kept);
            }
            slots_layout<G, true>(S, A, K, valid, x.ka, g);
            const int32_t znew = draw_block<G, false, true>(M, S, A, Rf, x, zo, valid, kept < 256, st, g);
            if (valid) zz[q] = (uint16_t)znew;
        }
        budget -= t1 - next;
        next = t1;
        if (next == kept) {
            // the sweep is complete
            if (s > F.burn_in) {
                for (int32_t j = g; j < S.L; j += G) {
                    const int32_t k = topic_of(S, j);
                    const uint32_t c = count_of(S, k);
                    if (c) atomicAdd(&acc[k], c);
                }
            }
            done = s;
            next = 0;
        }
    }
    if (g == 0) {
        F.prog[2 * sid] = done;
        F.prog[2 * sid + 1] = next;
    }
    __threadfence();
    if (done == F.sweeps) {
        const double denom = (double)kept + F.A;
        const double ns = (double)(F.sweeps - F.burn_in);
        float *theta = F.theta + (acc - F.acc);
        for (int32_t k = g; k < K; k += G)
            theta[k] = (float)(((double)acc[k] / ns + M.alpha[k]) / denom);
        double part = 0.0;
        for (int32_t q = g; q < kept; q += G) part += log((double)phi_at(M, wds[q], zz[q]));
        // (topics in a fixed order, whatever the slots)
        for (int32_t k = g; k < K; k += G) {
            const int32_t c = (int32_t)count_of(S, k);
            if (c > 0) {
                if constexpr (SYM) part += M.lg_alpha[c];
                else part += lgamma((double)c + M.alpha[k]) - lgamma(M.alpha[k]);
            }
        }
        const double tot = group_bcast_f64<G>(group_scan_incl<G>(part), G - 1);
        if (g == 0) F.ll[sid] = tot + M.lg_A[kept];
        // the step number last, once theta and ll are written (the group is
        // one wave: the fence orders every lane's writes before it)
        __threadfence();
        if (g == 0) F.fin[sid] = F.step_no;
    }
}

// one group's layout of a launch, and of its groups of 64 lanes (beside groups of
// 32, for what is not likely to fit those: the first blocks)
struct GroupLds {
    SlotLds own, wide;
};

template <int G, bool SYM, int W>
__global__ void __launch_bounds__(256, W) foldin_step_kernel(DevModel M, DevFoldin F, const int32_t *active,
                                                          int32_t n_active, GroupLds A)
{
    extern __shared__ __align__(16) uint8_t f_lds[];
    // the block's copy of fp32(R_k), then the groups' regions
    float *R = (float *)f_lds;
    for (int32_t k = threadIdx.x; k < M.K; k += blockDim.x) R[k] = (float)M.Rd[k];
    __syncthreads();
    uint8_t *base = f_lds + (M.K * 4 + 15) / 16 * 16;
    const int waves = (int)(blockDim.x >> 6), wave = (int)(threadIdx.x >> 6);
    const int32_t wide_blocks = G == 32 ? (F.n_wide + waves - 1) / waves : 0;
    if (G == 32 && (int32_t)blockIdx.x < wide_blocks) {
        const int32_t i = (int32_t)blockIdx.x * waves + wave;
        if (i < F.n_wide) foldin_slot<64, SYM>(M, F, active[i], R, base + wave * A.wide.group_bytes, A.wide);
        return;
    }
    const int slot = wave * (64 / G) + (int)(__lane_id() / G);   // group in the block
    const int32_t i = (G == 32 ? F.n_wide : 0) + ((int32_t)blockIdx.x - wide_blocks) * (waves * (64 / G)) + slot;
    if (i < n_active) foldin_slot<G, SYM>(M, F, active[i], R, base + slot * A.own.group_bytes, A.own);
}

// Launch of a kernel with groups of G lanes (wide: some of 64 lanes), their slots
// in LDS behind the block's copy of R_k: four waves a block, or as many as LDS
// holds.  go(waves, LDS bytes)
template <typename Launch>
static hipError_t launch_groups(int32_t K, int32_t G, bool wide, const GroupLds &A, Launch go)
{
    for (int waves = 4; waves >= 1; waves >>= 1) {
        size_t groups = (size_t)waves * (64 / G) * A.own.group_bytes;
        if (wide && groups < (size_t)waves * A.wide.group_bytes) groups = (size_t)waves * A.wide.group_bytes;
        const size_t lds = (size_t)(K * 4 + 15) / 16 * 16 + groups;
        if (lds > LDS_BYTES) continue;
        go(waves, lds);
        return hipGetLastError();
    }
    return hipErrorInvalidConfiguration;  // a wave's LDS exceeds the CU's
}

hipError_t launch_foldin_step(const DevModel &m, const DevFoldin &f, const int32_t *active, int32_t n_active,
                              int32_t n_cu, hipStream_t s)
{
    if (n_active == 0) return hipSuccess;
    const int32_t group = f.group;
    const GroupLds A = {slot_lds(group, m.K, f.max_len), slot_lds(64, m.K, f.wide_len)};
    return launch_groups(m.K, group, f.n_wide > 0, A, [&](int waves, size_t lds) {
        const int32_t per = waves * (64 / group);
        const int32_t blocks = (f.n_wide + waves - 1) / waves + (n_active - f.n_wide + per - 1) / per;
#define PULDA_FOLDIN(G_, S_, W_) foldin_step_kernel<G_, S_, W_><<<blocks, 64 * waves, lds, s>>>(m, f, active, n_active, A)
        const bool four = group == 64 && fits_at_four_only(blocks, n_cu);
        if (m.lg_alpha) {
            if (four) PULDA_FOLDIN(64, true, 4);
            else if (group == 64) PULDA_FOLDIN(64, true, 3);
            else if (group == 32) PULDA_FOLDIN(32, true, 3);
            else PULDA_FOLDIN(16, true, 3);
        } else {
            if (four) PULDA_FOLDIN(64, false, 4);
            else if (group == 64) PULDA_FOLDIN(64, false, 3);
            else if (group == 32) PULDA_FOLDIN(32, false, 3);
            else PULDA_FOLDIN(16, false, 3);
        }
#undef PULDA_FOLDIN
    });
}

// ---------------------------------------------------------------------------
// Held-out log-likelihood of new documents, log p(w_d | Phi, alpha), by the
// left-to-right algorithm of Wallach, Murray, Salakhutdinov and Mimno, the
// estimator behind the held-out comparison of Section 4.  One group of G
// lanes per (document, particle).  Tokens whose word is >= V or whose Phi
// column is empty are dropped; at step n (n = 0 .. nk - 1) the particle
// redraws its topics z_0 .. z_{n-1} in order, each from the token
// conditional of Section 3.5 given its other topics among the first n (the
// fold-in draw), then draws z_n from that conditional given z_<n and keeps
// its normaliser Z_n = sigma_a(w_n) + sigma_b(w_n).  A second kernel forms
// sum_n log((1/R) sum_r Z_n^(r) / (n + A)).  Draws use Philox counter
// (q, n, request, TAG_LTR + 256 r) for token q at step n (q = n: the new
// token).
// ---------------------------------------------------------------------------
template <int G>
__device__ __forceinline__ void ltr_particle(const DevModel &M, const DevHeldout &H, int64_t d, int32_t r,
                                             const float *Rf, uint8_t *lds, const SlotLds &A)
{
    SlotDoc S = slot_doc(lds, A);
    const int lane = __lane_id();
    const int g = lane & (G - 1);
    const int64_t s = H.doc_off[d];
    const int32_t len = (int32_t)(H.doc_off[d + 1] - s);
    const int64_t base = s * H.R + (int64_t)r * len;
    int32_t *kw = H.kw + base;
    uint16_t *zz = H.z + base;
    double *Zs = H.Zs + base;
    const uint32_t req = H.req[d];
    const uint32_t tag = TAG_LTR + ((uint32_t)r << 8);
    // kept tokens, in order
    int32_t nk = 0;
    for (int32_t p0 = 0; p0 < len; p0 += G) {
        const int32_t p = p0 + g;
        int32_t v = -1;
        bool keep = false;
        if (p < len) {
            v = H.words[s + p];
            keep = v >= 0 && v < M.V && M.colptr[v + 1] > M.colptr[v];
        }
        const uint64_t bal = group_ballot<G>(keep);
        if (keep) kw[nk + __builtin_popcountll(bal & ((1ull << g) - 1ull))] = v;
        nk += __builtin_popcountll(bal);
    }
    if (r == 0 && g == 0) H.kept[d] = nk;
    __threadfence();
    slots_load<G, false>(S, A, zz, 0, 0, g);
    ZStat st;
    for (int32_t n = 0; n < nk; ++n) {
        // redraw z_0 .. z_{n-1} in order, then draw z_n: blocks of G tokens,
        // lane q mod G holding token q.  (n tokens counted: the redraws may
        // settle the a-part at staging; only the new token's draw needs its Z)
        for (int32_t q0 = 0; q0 <= n; q0 += G) {
            const int32_t q = q0 + g;
            const bool redraw = q < n;
            int32_t zo = 0;
            LaneTok x = no_token();
            if (q <= n) {
                zo = redraw ? zz[q] : 0;
                const r4 rr = philox((uint32_t)q, (uint32_t)n, req, tag, H.key0, H.key1);
                x = stage_token(M, kw[q], zo, rr, redraw ? n : 0);
            }
            slots_layout<G, true>(S, A, M.K, q <= n, x.ka, g);
            int32_t znew = draw_block<G, false, true>(M, S, A, Rf, x, zo, redraw, nk < 256, st, g);
            if (n - q0 < G) {
                // the new token, from the counts of z_<n in fp64 (its Z)
                const int c = n - q0;
                const int32_t v = group_bcast<G>(x.v, c);
                const float u0 = __int_as_float(group_bcast<G>(__float_as_int(x.u0), c));
                const int32_t ka = group_bcast<G>(x.ka, c);
                double Z;
                auto count = [&](int32_t, int32_t k) { return count_of(S, k); };
                int32_t at;
                if (S.dense) at = column_draw_f64<G>(M, S, v, u0, Z);
                else at = slots_draw_f64<G>(M, S, v, u0, (S.L + G - 1) / G, count, Z);
                const int32_t k = at < 0 ? ka : topic_of(S, at);
                if (g == 0) {
                    // (its bit may have been dropped with the block's counts)
                    set_count(S, k, count_of(S, k) + 1);
                    S.P[k >> 5] |= 1u << (k & 31);
                    Zs[n] = Z;
                }
                if (g == c) znew = k;
                lds_order();
            }
            if (q <= n) zz[q] = (uint16_t)znew;
        }
    }
}

// The particles of a document read the same words' rows again and again, so its
// blocks are put on one XCD (block b runs on XCD b mod 8), beside few other
// documents: document j of a launch's part on XCD j mod 8, in order.  With parts
// of fewer than LTR_SPREAD documents blocks follow each other (one document's
// would fill one XCD only).  2,000 documents of up to 500 tokens, 10 particles,
// Algorithm 1's Phi (4 KB a row): 438 ms on 64 lanes, 398 so; the urn's 132 and 124.
constexpr int64_t LTR_SPREAD = 64;
constexpr int32_t XCDS = 8;

// blocks of `per` particles for n documents
__host__ __device__ inline int64_t ltr_blocks(int64_t n, int64_t R, int64_t per)
{
    return n < LTR_SPREAD ? (n * R + per - 1) / per : XCDS * (((n + XCDS - 1) / XCDS * R + per - 1) / per);
}

// document and particle of group `slot` of block b; false: none
__device__ __forceinline__ bool ltr_work(int64_t n, int32_t R, int32_t per, int64_t b, int slot, int64_t &j, int32_t &r)
{
    const int64_t spread = n < LTR_SPREAD ? 1 : XCDS;
    const int64_t i = b / spread * per + slot;
    j = b % spread + spread * (i / R);
    r = (int32_t)(i % R);
    return j < n;
}

template <int G, int W>
__global__ void __launch_bounds__(256, W) ltr_kernel(DevModel M, DevHeldout H, GroupLds A)
{
    extern __shared__ __align__(16) uint8_t h_lds[];
    float *R = (float *)h_lds;
    for (int32_t k = threadIdx.x; k < M.K; k += blockDim.x) R[k] = (float)M.Rd[k];
    __syncthreads();
    uint8_t *base = h_lds + (M.K * 4 + 15) / 16 * 16;
    const int waves = (int)(blockDim.x >> 6), wave = (int)(threadIdx.x >> 6);
    const int64_t wide_blocks = G == 32 ? ltr_blocks(H.n_wide, H.R, waves) : 0;
    int64_t j;
    int32_t r;
    if (G == 32 && (int64_t)blockIdx.x < wide_blocks) {
        if (ltr_work(H.n_wide, H.R, waves, blockIdx.x, wave, j, r))
            ltr_particle<64>(M, H, H.order[j], r, R, base + wave * A.wide.group_bytes, A.wide);
        return;
    }
    const int slot = wave * (64 / G) + (int)(__lane_id() / G);   // group in the block
    if (ltr_work(H.D - H.n_wide, H.R, waves * (64 / G), (int64_t)blockIdx.x - wide_blocks, slot, j, r))
        ltr_particle<G>(M, H, H.order[H.n_wide + j], r, R, base + slot * A.own.group_bytes, A.own);
}

// one wave per document: sum over steps of log((1/R) sum_r Z_n^(r) / (n + A)),
// the particles added in ascending order
__global__ void __launch_bounds__(256) ltr_finish_kernel(DevHeldout H)
{
    const int64_t d = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (d >= H.D) return;
    const int lane = __lane_id();
    const int64_t s = H.doc_off[d];
    const int32_t len = (int32_t)(H.doc_off[d + 1] - s);
    const int32_t nk = H.kept[d];
    double part = 0.0;
    for (int32_t n = lane; n < nk; n += 64) {
        double sum = 0.0;
        for (int32_t r = 0; r < H.R; ++r) sum += H.Zs[s * H.R + (int64_t)r * len + n] / ((double)n + H.A);
        part += log(sum / (double)H.R);
    }
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if (lane == 0) H.ll[d] = part;
}

hipError_t launch_heldout(const DevModel &m, const DevHeldout &h, hipStream_t s)
{
    if (h.D == 0) return hipSuccess;
    const int32_t group = h.group;
    const GroupLds A = {slot_lds(group, m.K, h.longest), slot_lds(64, m.K, h.wide_len)};
    hipError_t e = launch_groups(m.K, group, h.n_wide > 0, A, [&](int waves, size_t lds) {
        const unsigned blocks = (unsigned)(ltr_blocks(h.n_wide, h.R, waves) + ltr_blocks(h.D - h.n_wide, h.R, waves * (64 / group)));
        // (phi's own rows, Algorithm 1's: 227 ms with 128 registers, 264 with
        // 168, at the sizes of ltr_blocks; the urn's 140 and 134)
        if (group == 64) ltr_kernel<64, 3><<<blocks, 64 * waves, lds, s>>>(m, h, A);
        else if (group == 32 && m.values) ltr_kernel<32, 4><<<blocks, 64 * waves, lds, s>>>(m, h, A);
        else if (group == 32) ltr_kernel<32, 3><<<blocks, 64 * waves, lds, s>>>(m, h, A);
        else ltr_kernel<16, 3><<<blocks, 64 * waves, lds, s>>>(m, h, A);
    });
    if (e != hipSuccess) return e;
    ltr_finish_kernel<<<(unsigned)((h.D + 3) / 4), 256, 0, s>>>(h);
    return hipGetLastError();
}

}  // namespace pulda
