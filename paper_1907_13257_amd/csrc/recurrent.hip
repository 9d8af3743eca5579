// recurrent.hip -- the sequential part of the LSTM step for the layers that do
// not fit the XCD-local kernels (fp32 storage, LSTMP, bf16 cells wider than
// 1024 or more than 512 rows) and have a tiling here (up to 4096 cells): one
// persistent, cooperatively launched kernel for the forward
// recurrence and one for back-propagation through time.
//
// Ownership.  Workgroup (ht, bg) owns the cells j in [ht*HN, ht*HN + HN) for
// the batch tiles bt = bg, bg + bgroups, ...  Forward: it keeps the 4*HN rows
// of R that feed its cells (cell-major: row 4u + g is gate g of cell u) in LDS
// for the whole kernel and, per step, multiplies h_{t-1} of its batch rows by
// them on the matrix cores, adds the precomputed input projection and applies
// the cell update.  Backward: it keeps the HN columns of R (rows of R^T) for
// its cells and computes, per step, the gate gradients of its cells and then
// their share of dh_{t-1} = R^T dz.  The projections of LSTMP (h = P m, and
// R^T dz into the projected carry) reduce over every cell: their 16-column
// blocks are dealt to the workgroups of a batch group.
//
// Exchange.  Only the workgroups of one batch group depend on each other.  A
// step's exchanged rows (y, m, dz, dH) are written with device-coherent (sc1)
// stores and read with sc1 loads, so no cache needs a write-back or an
// invalidate; every element is written once and read after the step's flags.
// A workgroup waits for its own stores, then stores the step's number into its
// flag word; one wave of every consumer polls the group's flag words.  With
// fences at agent scope around one counter (an L2 write-back and invalidate per
// workgroup) a step barrier over 256 workgroups took 24.5 us; here a whole step
// of a 64-cell fp32 layer takes about 2 us.  Per step, before and after: fp32
// H = 1024 at 32 rows 40.5 -> 5.7 us forward, 68 -> 13.8 us backward; LSTMP
// H = 1024, Hp = 512 at 64 rows 74 -> 10.7 us and 73 -> 13.7 us.
//
// Products.  The eight waves split k; a wave reads the exchanged rows straight
// into MFMA operand registers (each element once per workgroup), eight 64-byte
// chunks of k in flight while the previous eight are multiplied (four with 64
// rows per tile; four or two where the weights stream as well), so a product
// is bound by the rows' bytes and not by one memory latency per chunk (f32,
// H = 1024, K = 4096: one chunk in flight took 64 us per step).  The eight
// partial sums meet in LDS.
//
// Every wait has a wall-clock watchdog: on expiry it raises an abort word (so
// every other workgroup leaves too) and a sticky error word of the library (a
// device variable, zero at load) that the host reads and clears with
// lstm_check.
#include "device_common.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <cstdlib>

namespace lstm355 {

__device__ unsigned g_watchdog_tripped = 0;

namespace {

constexpr int WGT = 512;                 // 8 waves, 2 per SIMD
constexpr int NWAVE = WGT / 64;
constexpr unsigned OOB_OFFSET = 0x80000000u;

// Device-coherent stores of exchanged values.
__device__ __forceinline__ void store_coherent(bf16_t *p, bf16_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_coherent(float *p, float v)
{
    __hip_atomic_store(reinterpret_cast<unsigned *>(p), __float_as_uint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// The flag words of one batch group (n workgroups, this one is `me`).
struct GroupSync {
    unsigned *flags, *abort;
    int n, me;
    unsigned long long timeout;

    // Everything this workgroup stored before is visible to whoever sees `epoch`.
    __device__ __forceinline__ void signal(unsigned epoch) const
    {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) __hip_atomic_store(flags + me, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // Waits until every workgroup of the group has signalled `epoch`; false
    // (in every thread) if the watchdog expired or another workgroup gave up.
    __device__ __forceinline__ bool wait(unsigned epoch, int *s_abort) const
    {
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc(flags, (short)0, n * 4, 0x00020000);
            const unsigned long long t0 = wall_clock64();
            while (true) {
                const u32x4 v =
                    __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rf, lane * 16, 0, 16));
                bool ready = true;
#pragma unroll
                for (int i = 0; i < 4; ++i) ready = ready && (lane * 4 + i >= n || v[i] >= epoch);
                if (__builtin_amdgcn_ballot_w64(!ready) == 0) break;
                const unsigned ab = __hip_atomic_load(abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (ab != 0 || wall_clock64() - t0 > timeout) {
                    if (lane == 0) {
                        if (ab == 0) {
                            __hip_atomic_fetch_or(&g_watchdog_tripped, TRIP_WATCHDOG, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                            __hip_atomic_store(abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                        *s_abort = 1;
                    }
                    break;
                }
            }
        }
        __syncthreads();
        return *s_abort == 0;
    }
};

// acc[i][j] += (weight rows of block j) x (16 batch rows of block i) over this
// wave's k chunks [c0, c1) of 64 bytes: the transposed product, so lane l ends
// with batch row l % 16 and weight rows 4*(l / 16) .. +3 of the block.
//   ra, aoff: exchanged rows, read with sc1 loads; aoff[i] is the byte offset
//     of this lane's row (OOB_OFFSET and up: a row past the end, zero).
//   w, woff: weights, woff[j] the byte offset of this lane's row; WLDS: in LDS,
//     zero-padded to whole chunks; else in global memory (negative: zero).
template <typename TI, int MB, int NB, bool WLDS>
__device__ __forceinline__ void wave_product(__amdgpu_buffer_rsrc_t ra, const unsigned (&aoff)[MB], int kbytes,
                                             int c0, int c1, const char *w, const long (&woff)[NB],
                                             f32x4 (&acc)[MB][NB])
{
    // chunks per batch, two batches in flight
    constexpr int U = WLDS ? (MB >= 4 ? 4 : 8) : (MB * NB >= 4 ? 2 : 4);
    constexpr int UW = WLDS ? 1 : U;
    const int kl = ((threadIdx.x & 63) >> 4) * 16;
    struct Batch {
        u32x4 a[U][MB], w[UW][NB];
    };
    auto load = [&](int c, Batch &f) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kb = (c + u) * 64 + kl;
            const bool in = c + u < c1 && kb < kbytes;
#pragma unroll
            for (int i = 0; i < MB; ++i)
                f.a[u][i] = __builtin_bit_cast(
                    u32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, in ? aoff[i] + kb : OOB_OFFSET, 0, 16));
            if constexpr (!WLDS) {
#pragma unroll
                for (int j = 0; j < NB; ++j) f.w[u][j] = in && woff[j] >= 0 ? ldg16(w + woff[j] + kb) : zero16();
            }
        }
    };
    auto multiply = [&](int c, const Batch &f) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c + u >= c1) break;   // wave-uniform
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                u32x4 fw;
                if constexpr (WLDS)
                    fw = *reinterpret_cast<const u32x4 *>(w + (int)woff[j] + (c + u) * 64 + kl);
                else
                    fw = f.w[u][j];
#pragma unroll
                for (int i = 0; i < MB; ++i) mfma16(acc[i][j], fw, f.a[u][i], TI{});
            }
        }
    };
    if (c0 >= c1) return;
    Batch f0, f1;
    load(c0, f0);
    for (int c = c0; c < c1; c += 2 * U) {
        if (c + U < c1) load(c + U, f1);
        multiply(c, f0);
        if (c + U < c1) {
            if (c + 2 * U < c1) load(c + 2 * U, f0);
            multiply(c + U, f1);
        }
    }
}

// One tile's product: rows [b0, b0 + 16 MB) of A (row b of the exchanged
// matrix at A + b*lda elements, K wide) times 16*NB weight rows, the eight
// waves' partial sums left in red[wave][row][16 NB + 4] (no barrier after).
template <typename TI, int MB, int NB>
__device__ __forceinline__ void tile_product(const char *A, long lda, int b0, int B, int K, const char *w,
                                             const long (&woff)[NB], bool wlds, float *red)
{
    constexpr int BM = 16 * MB, RP = 16 * NB + 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kbytes = K * (int)sizeof(TI);
    const int nkc = (kbytes + 63) / 64, per = (nkc + NWAVE - 1) / NWAVE;
    const int c0 = min(nkc, wave * per), c1 = min(nkc, c0 + per);
    const int nrow = min(BM, B - b0);
    const long rowb = lda * (long)sizeof(TI);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(A) + (long)b0 * rowb, (short)0, (int)((nrow - 1) * rowb + kbytes), 0x00020000);
    unsigned aoff[MB];
    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int r = i * 16 + (lane & 15);
        aoff[i] = r < nrow ? (unsigned)(r * rowb) : OOB_OFFSET;
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (wlds)
        wave_product<TI, MB, NB, true>(ra, aoff, kbytes, c0, c1, w, woff, acc);
    else
        wave_product<TI, MB, NB, false>(ra, aoff, kbytes, c0, c1, w, woff, acc);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
            *reinterpret_cast<f32x4 *>(red + (wave * BM + i * 16 + (lane & 15)) * RP + j * 16 + 4 * (lane >> 4)) =
                acc[i][j];
}

// Sum of the eight partials of one output (row, column) of a tile product.
template <int BM, int RP>
__device__ __forceinline__ float red_sum(const float *red, int row, int col)
{
    float v = 0.0f;
#pragma unroll
    for (int q = 0; q < NWAVE; ++q) v += red[(q * BM + row) * RP + col];
    return v;
}

// Rows [0, 16 NB) of a weight slice into LDS: row n from src(n) (NULL: zeros),
// zero-padded to whole 64-byte chunks of k.
template <typename F>
__device__ __forceinline__ void load_slice(char *dst, int pitch, int nrows, int kbytes, F src)
{
    const int vpr = (kbytes + 63) / 64 * 4;   // 16-byte vectors per row
    for (int idx = threadIdx.x; idx < nrows * vpr; idx += WGT) {
        const int n = idx / vpr, kv = idx % vpr;
        const char *p = src(n);
        *reinterpret_cast<u32x4 *>(dst + n * pitch + kv * 16) = p && kv * 16 < kbytes ? ldg16(p + kv * 16) : zero16();
    }
}

// The share of a projection's output that a workgroup of a batch group
// computes: 16-column blocks of N columns.  With at least as many workgroups
// as blocks each takes one block (its weights stay in LDS where they fit) and
// every nper-th batch tile of the group from tile index `part`; else each
// takes every nHT-th block and all tiles.
struct Deal {
    int nb, nb_step, nbn, part, nper;
    __device__ __forceinline__ Deal(int ht, int nHT, int N)
    {
        nbn = (N + 15) / 16;
        if (nHT >= nbn) {
            nper = nHT / nbn;
            nb = ht % nbn;
            part = ht / nbn;
            nb_step = nbn;
            if (part >= nper) nb = nbn;   // surplus workgroups have no share
        } else {
            nper = 1;
            part = 0;
            nb = ht;
            nb_step = nHT;
        }
    }
};

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
struct FwdArgs {
    int T, B, H, Hp, Hr, reverse;
    long ldy;
    const char *R, *P, *h0;
    const float *c0;
    float *gates, *cs;
    char *ms, *y, *hT;
    float *cT;
    unsigned *sync;
    unsigned long long timeout;
    int nHT, nBT, bgroups, w_lds, p_lds, kpitch, ppitch;
};

// MB blocks of 16 batch rows per tile, NB blocks of 16 gate rows: HN = 4*NB
// cells.  At most one cell per thread (MB*NB <= 4 blocks of 64 cells).
template <typename TI, int MB, int NB, bool PROJ>
__global__ __launch_bounds__(WGT) void lstm_fwd_kernel(FwdArgs a)
{
    constexpr int BM = 16 * MB, NT = 16 * NB, HN = 4 * NB, RP = NT + 4, RPP = 20;
    constexpr int REDF = NWAVE * BM * (RP > RPP ? RP : RPP);
    static_assert(BM * HN <= WGT, "one cell per thread");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ int s_abort;
    float *red = reinterpret_cast<float *>(lds);
    char *rs = lds + REDF * 4;                               // [NT][kpitch] when w_lds
    char *ps = rs + (a.w_lds ? NT * a.kpitch : 0);           // [16][ppitch] when p_lds

    const int tid = threadIdx.x, lane = tid & 63;
    const int ht = blockIdx.x % a.nHT, bg = blockIdx.x / a.nHT;
    const int j0 = ht * HN;
    const int H = a.H, Hr = a.Hr, B = a.B;
    const long G4 = 4L * H;
    const long es = (long)sizeof(TI);
    const GroupSync gs{a.sync + SYNC_FLAGS + bg * ((a.nHT + 3) & ~3), a.sync + SYNC_ABORT, a.nHT, ht, a.timeout};
    if (tid == 0) s_abort = 0;

    // gate row n of the slice: gate n % 4 of cell n / 4
    auto rrow = [&](int n) -> const char * {
        const int j = j0 + (n >> 2);
        return j < H ? a.R + ((long)(n & 3) * H + j) * Hr * es : nullptr;
    };
    long woff[NB];
    if (a.w_lds) load_slice(rs, a.kpitch, NT, Hr * (int)es, rrow);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int n = j * 16 + (lane & 15);
        const char *p = rrow(n);
        woff[j] = a.w_lds ? (long)n * a.kpitch : (p ? p - a.R : -1L);
    }
    const Deal dl(ht, a.nHT, PROJ ? a.Hp : 16);
    if (PROJ && a.p_lds && dl.nb < dl.nbn)
        load_slice(ps, a.ppitch, 16, H * (int)es, [&](int n) -> const char * {
            const int p = dl.nb * 16 + n;
            return p < a.Hp ? a.P + (long)p * H * es : nullptr;
        });
    __syncthreads();

    const int bl = tid / HN, u = tid % HN, j = j0 + u;
    const bool single = a.nBT <= a.bgroups;                  // one tile per workgroup: c stays in a register
    float creg = 0.0f;
    unsigned epoch = 0;
    int tprev = -1;
    for (int s = 0; s < a.T; ++s) {
        const int t = a.reverse ? a.T - 1 - s : s;
        const char *hprev = s == 0 ? a.h0 : a.y + (long)tprev * B * a.ldy * es;
        const long ldh = s == 0 ? Hr : a.ldy;
        const bool last = s == a.T - 1;

        for (int bt = bg; bt < a.nBT; bt += a.bgroups) {
            const int b0 = bt * BM, b = b0 + bl;
            const bool has = tid < BM * HN && b < B && j < H;
            // the cell's input projection and previous state travel during the wait and the product
            const long row = (long)t * B + b;
            float z[4], cp = creg;
#pragma unroll
            for (int g = 0; g < 4; ++g) z[g] = has ? a.gates[row * G4 + (long)g * H + j] : 0.0f;
            if (s == 0)
                cp = has && a.c0 ? a.c0[(long)b * H + j] : 0.0f;
            else if (!single)
                cp = has ? a.cs[((long)tprev * B + b) * H + j] : 0.0f;
            if (s > 0 && bt == bg && !gs.wait(epoch, &s_abort)) return;
            if (hprev) {
                tile_product<TI, MB, NB>(hprev, ldh, b0, B, Hr, a.w_lds ? rs : a.R, woff, a.w_lds != 0, red);
                __syncthreads();
            }
            if (has) {
                if (hprev) {
#pragma unroll
                    for (int q = 0; q < NWAVE; ++q) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(red + (q * BM + bl) * RP + 4 * u);
#pragma unroll
                        for (int g = 0; g < 4; ++g) z[g] += v[g];
                    }
                }
                const float ig = sigmoid_f(z[0]), fg = sigmoid_f(z[1]), gg = tanh_f(z[2]), og = sigmoid_f(z[3]);
                const float c = fg * cp + ig * gg;
                const TI mv = from_f32<TI>(og * tanh_f(c));
                creg = c;
                if (PROJ) {
                    store_coherent(reinterpret_cast<TI *>(a.ms) + row * H + j, mv);
                } else {
                    store_coherent(reinterpret_cast<TI *>(a.y) + row * a.ldy + j, mv);
                    if (last && a.hT) reinterpret_cast<TI *>(a.hT)[(long)b * Hr + j] = mv;
                }
                float *gp = a.gates + row * G4 + j;
                gp[0] = ig;
                gp[H] = fg;
                gp[2 * H] = gg;
                gp[3 * H] = og;
                a.cs[row * H + j] = c;
                if (last && a.cT) a.cT[(long)b * H + j] = c;
            }
            __syncthreads();   // red is rewritten by the next tile or product
        }

        if (PROJ) {
            // h_t = P m_t needs every cell's m_t
            gs.signal(++epoch);
            if (!gs.wait(epoch, &s_abort)) return;
            const char *mt = a.ms + (long)t * B * H * es;
            TI *yt = reinterpret_cast<TI *>(a.y) + (long)t * B * a.ldy;
            for (int nb = dl.nb; nb < dl.nbn; nb += dl.nb_step) {
                const int pr = nb * 16 + (lane & 15);
                const long poff[1] = {a.p_lds ? (long)(lane & 15) * a.ppitch : (pr < a.Hp ? (long)pr * H * es : -1L)};
                for (int bt = bg + dl.part * a.bgroups; bt < a.nBT; bt += dl.nper * a.bgroups) {
                    const int b0 = bt * BM;
                    tile_product<TI, MB, 1>(mt, H, b0, B, H, a.p_lds ? ps : a.P, poff, a.p_lds != 0, red);
                    __syncthreads();
                    for (int e = tid; e < BM * 16; e += WGT) {
                        const int b = b0 + e / 16, p = nb * 16 + e % 16;
                        if (b >= B || p >= a.Hp) continue;
                        const TI hv = from_f32<TI>(red_sum<BM, RPP>(red, e / 16, e % 16));
                        store_coherent(yt + (long)b * a.ldy + p, hv);
                        if (last && a.hT) reinterpret_cast<TI *>(a.hT)[(long)b * Hr + p] = hv;
                    }
                    __syncthreads();
                }
            }
        }
        if (!last) gs.signal(++epoch);
        tprev = t;
    }
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
struct BwdArgs {
    int T, B, H, Hp, Hr, reverse;
    long ldy;
    const char *Rt, *Pt, *dy, *dhT;
    const float *dcT, *c0, *gates, *cs;
    char *dz, *dH, *dh0;
    float *dc0;
    float *dcn, *dhn;       // per-cell carries [B][H] (several tiles per workgroup)
    float *dbpart;          // [bgroups][4H] bias gradients per batch group
    unsigned *sync;
    unsigned long long timeout;
    int HN, nHT, nBT, bgroups, w_lds, p_lds, kpitch, ppitch;
};

// The weight slice of the workgroup's cells is HN (<= 16) rows of R^T, or of
// P^T for LSTMP; lanes past HN repeat its rows and their outputs are dropped.
// At most one cell per thread (16*MB*HN <= 512).
template <typename TI, int MB, bool PROJ>
__global__ __launch_bounds__(WGT) void lstm_bwd_kernel(BwdArgs a)
{
    constexpr int BM = 16 * MB, RP = 20;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ int s_abort;
    float *red = reinterpret_cast<float *>(lds);             // [8][BM][RP], at the end [BM][HN][4]
    char *ws = lds + NWAVE * BM * RP * 4;                    // [HN][kpitch] when w_lds

    const int tid = threadIdx.x, lane = tid & 63;
    const int HN = a.HN;
    const int ht = blockIdx.x % a.nHT, bg = blockIdx.x / a.nHT;
    const int j0 = ht * HN;
    const int H = a.H, Hr = a.Hr, B = a.B, Hp = a.Hp;
    const long G4 = 4L * H;
    const long es = (long)sizeof(TI);
    const int Kw = PROJ ? Hp : 4 * H;                        // k extent of the slice
    const char *wsrc = PROJ ? a.Pt : a.Rt;                   // rows j of P^T or R^T
    char *ps = ws + (a.w_lds ? HN * a.kpitch : 0);           // [16][ppitch] when p_lds: R^T rows of the share
    const GroupSync gs{a.sync + SYNC_FLAGS + bg * ((a.nHT + 3) & ~3), a.sync + SYNC_ABORT, a.nHT, ht, a.timeout};
    if (tid == 0) s_abort = 0;

    if (a.w_lds)
        load_slice(ws, a.kpitch, HN, Kw * (int)es,
                   [&](int n) -> const char * { return j0 + n < H ? wsrc + (long)(j0 + n) * Kw * es : nullptr; });
    const int wn = (lane & 15) % HN;
    const long woff[1] = {a.w_lds ? (long)wn * a.kpitch : (j0 + wn < H ? (long)(j0 + wn) * Kw * es : -1L)};
    const Deal dl(ht, a.nHT, PROJ ? Hp : 16);
    if (PROJ && a.p_lds && dl.nb < dl.nbn)
        load_slice(ps, a.ppitch, 16, (int)(G4 * es), [&](int n) -> const char * {
            const int p = dl.nb * 16 + n;
            return p < Hp ? a.Rt + (long)p * G4 * es : nullptr;
        });
    unsigned epoch = 0;

    if (PROJ) {
        // dh of the first visited step (in reverse order): dy + dhT, the group's rows
        const int t = a.reverse ? 0 : a.T - 1;
        TI *dHt = reinterpret_cast<TI *>(a.dH) + (long)t * B * Hp;
        const TI *dyt = reinterpret_cast<const TI *>(a.dy) + (long)t * B * a.ldy;
        const TI *dhT = reinterpret_cast<const TI *>(a.dhT);
        for (int bt = bg; bt < a.nBT; bt += a.bgroups)
            for (int i = ht * WGT + tid; i < BM * Hp; i += a.nHT * WGT) {
                const long b = bt * BM + i / Hp, p = i % Hp;
                if (b >= B) continue;
                float v = to_f32(dyt[b * a.ldy + p]);
                if (dhT) v += to_f32(dhT[b * Hp + p]);
                store_coherent(dHt + b * Hp + p, from_f32<TI>(v));
            }
        gs.signal(++epoch);
    } else {
        __syncthreads();
    }

    const int bl = tid / HN, u = tid % HN, j = j0 + u;
    const bool cell = tid < BM * HN && j < H;
    const bool single = a.nBT <= a.bgroups;                  // one tile per workgroup: carries stay in registers
    float dcreg = 0.0f, dhreg = 0.0f;
    float dbacc[4] = {0.f, 0.f, 0.f, 0.f};                   // this thread's rows, summed over tiles and steps
    for (int s = a.T - 1; s >= 0; --s) {
        const int t = a.reverse ? a.T - 1 - s : s;
        const int tp = a.reverse ? t + 1 : t - 1;            // previously visited step in the forward order
        const bool first = s == a.T - 1;

        for (int bt = bg; bt < a.nBT; bt += a.bgroups) {
            const int b0 = bt * BM, b = b0 + bl;
            const bool has = cell && b < B;
            const long row = (long)t * B + b, cidx = (long)b * H + j;
            float gv[4], c = 0.0f, cp = 0.0f, dm = 0.0f, dcin = dcreg;
#pragma unroll
            for (int g = 0; g < 4; ++g) gv[g] = has ? a.gates[row * G4 + (long)g * H + j] : 0.0f;
            if (has) {
                c = a.cs[row * H + j];
                cp = s == 0 ? (a.c0 ? a.c0[cidx] : 0.0f) : a.cs[((long)tp * B + b) * H + j];
                if (first)
                    dcin = a.dcT ? a.dcT[cidx] : 0.0f;
                else if (!single)
                    dcin = a.dcn[cidx];
                if (!PROJ) {
                    dm = to_f32(reinterpret_cast<const TI *>(a.dy)[row * a.ldy + j]);
                    if (first)
                        dm += a.dhT ? to_f32(reinterpret_cast<const TI *>(a.dhT)[(long)b * Hr + j]) : 0.0f;
                    else
                        dm += single ? dhreg : a.dhn[cidx];
                }
            }
            if (PROJ) {
                // dm = P^T dh for this tile's rows and the workgroup's cells
                if (bt == bg && !gs.wait(epoch, &s_abort)) return;
                tile_product<TI, MB, 1>(a.dH + (long)t * B * Hp * es, Hp, b0, B, Hp, a.w_lds ? ws : wsrc, woff,
                                        a.w_lds != 0, red);
                __syncthreads();
                if (has) dm = red_sum<BM, RP>(red, bl, u);
            }
            if (has) {
                const float ig = gv[0], fg = gv[1], gg = gv[2], og = gv[3];
                const float tc = tanh_f(c);
                const float d_o = dm * tc;
                const float d_c = dcin + dm * og * (1.0f - tc * tc);
                const float d_i = d_c * gg, d_g = d_c * ig, d_f = d_c * cp;
                const float z[4] = {d_i * ig * (1.0f - ig), d_f * fg * (1.0f - fg), d_g * (1.0f - gg * gg),
                                    d_o * og * (1.0f - og)};
                TI *dz = reinterpret_cast<TI *>(a.dz) + row * G4 + j;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    store_coherent(dz + (long)g * H, from_f32<TI>(z[g]));
                    dbacc[g] += z[g];
                }
                dcreg = d_c * fg;
                if (!single) a.dcn[cidx] = dcreg;
                if (s == 0 && a.dc0) a.dc0[cidx] = dcreg;
            }
            if (PROJ) __syncthreads();   // red is rewritten by the next tile
        }

        // dh_{t-1} = R^T dz_t needs every cell's dz_t
        if (s == 0 && !a.dh0) break;
        gs.signal(++epoch);
        const char *dzt = a.dz + (long)t * B * G4 * es;
        if (PROJ) {
            if (!gs.wait(epoch, &s_abort)) return;
            TI *dHp = s > 0 ? reinterpret_cast<TI *>(a.dH) + (long)tp * B * Hp : nullptr;
            const TI *dyp = s > 0 ? reinterpret_cast<const TI *>(a.dy) + (long)tp * B * a.ldy : nullptr;
            for (int nb = dl.nb; nb < dl.nbn; nb += dl.nb_step) {
                const int pr = nb * 16 + (lane & 15);
                const long poff[1] = {a.p_lds ? (long)(lane & 15) * a.ppitch : (pr < Hp ? (long)pr * G4 * es : -1L)};
                for (int bt = bg + dl.part * a.bgroups; bt < a.nBT; bt += dl.nper * a.bgroups) {
                    const int b0 = bt * BM;
                    tile_product<TI, MB, 1>(dzt, G4, b0, B, (int)G4, a.p_lds ? ps : a.Rt, poff, a.p_lds != 0, red);
                    __syncthreads();
                    for (int e = tid; e < BM * 16; e += WGT) {
                        const long b = b0 + e / 16, p = nb * 16 + e % 16;
                        if (b >= B || p >= Hp) continue;
                        const float v = red_sum<BM, RP>(red, e / 16, e % 16);
                        if (dHp)
                            store_coherent(dHp + b * Hp + p, from_f32<TI>(v + to_f32(dyp[b * a.ldy + p])));
                        else
                            reinterpret_cast<TI *>(a.dh0)[b * Hp + p] = from_f32<TI>(v);
                    }
                    __syncthreads();
                }
            }
            if (s > 0) gs.signal(++epoch);
        } else {
            for (int bt = bg; bt < a.nBT; bt += a.bgroups) {
                const int b0 = bt * BM, b = b0 + bl;
                if (bt == bg && !gs.wait(epoch, &s_abort)) return;
                tile_product<TI, MB, 1>(dzt, G4, b0, B, (int)G4, a.w_lds ? ws : wsrc, woff, a.w_lds != 0, red);
                __syncthreads();
                if (cell && b < B) {
                    dhreg = red_sum<BM, RP>(red, bl, u);
                    if (s == 0)
                        reinterpret_cast<TI *>(a.dh0)[(long)b * Hr + j] = from_f32<TI>(dhreg);
                    else if (!single)
                        a.dhn[(long)b * H + j] = dhreg;
                }
                __syncthreads();   // red is rewritten by the next tile
            }
        }
    }
    // bias gradient: this workgroup's rows, in row order; one partial per batch group
    __syncthreads();
    if (tid < BM * HN) {
#pragma unroll
        for (int g = 0; g < 4; ++g) red[tid * 4 + g] = cell ? dbacc[g] : 0.0f;
    }
    __syncthreads();
    if (tid < 4 * HN) {
        const int g = tid / HN, uu = tid % HN;
        float v = 0.0f;
        for (int r = 0; r < BM; ++r) v += red[(r * HN + uu) * 4 + g];
        if (j0 + uu < H) a.dbpart[(long)bg * G4 + (long)g * H + j0 + uu] = v;
    }
}

// ---------------------------------------------------------------------------
// host side: tiling choice and launch
// ---------------------------------------------------------------------------
int g_lds_limit = 0;
unsigned long long g_timeout_ticks = 0;

void device_limits()
{
    if (g_lds_limit) return;
    int dev = 0, lds = 0, khz = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || lds <= 0)
        lds = 64 * 1024;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0) khz = 100000;
    g_lds_limit = lds;
    g_timeout_ticks = (unsigned long long)khz * 1000ull * 2ull;  // 2 seconds
}

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// LDS row pitch of a weight slice: whole 64-byte chunks of k plus 16 bytes, so
// that the 16 rows one fragment read touches start in distinct banks.
int slice_pitch(long k, size_t es) { return (int)(round_up((size_t)k * es, 64) + 16); }

// Cost of one tile product in nanoseconds: the larger of the matrix-core time
// and the exchanged rows at the rate one CU reads them while all do (about
// 30 bytes per ns), streamed weights at twice that rate, and a fixed part
// (latency, reduction through LDS, barriers).
double product_ns(int rows, int MB, int NB, double K, size_t es, bool wlds)
{
    const double chunks = K * (double)es / 64.0;
    const double mfma = MB * NB * chunks * (es == 4 ? 128.0 : 16.0) / 4.0 / 2.4;
    double mem = rows * K * (double)es / 30.0;
    if (!wlds) mem += 16.0 * NB * K * (double)es / 60.0;
    return std::max(mfma, mem) + 800.0;
}

constexpr double SYNC_NS = 2000.0;
constexpr int NVAR = 6;
constexpr int VAR_MB[NVAR] = {1, 1, 1, 2, 2, 4};
constexpr int VAR_NB[NVAR] = {1, 2, 4, 1, 2, 1};   // forward: blocks of 16 gate rows, HN = 4 NB; backward: HN = 4 NB too

}  // namespace

// Both directions choose the cells per workgroup (4, 8 or 16) and the batch
// rows per tile (16, 32, 64) that minimise the modelled time of a step.
static bool plan(bool fwd, DType t, const RecShape &sh, int num_cus, RecTiling *out)
{
    device_limits();
    const size_t es = dsize(t);
    const int Hr = sh.Hp ? sh.Hp : sh.H;
    const long Kw = fwd ? Hr : (sh.Hp ? sh.Hp : 4L * sh.H);      // k of the resident slice
    const long Kd = fwd ? sh.H : 4L * sh.H;                      // k of the projection (LSTMP)
    const long ldmax = std::max<long>(sh.ldy, 4L * sh.H);
    bool found = false;
    double best = 0;
    for (int v = 0; v < NVAR; ++v) {
        const int MB = VAR_MB[v], NB = VAR_NB[v], HN = 4 * NB, BM = 16 * MB;
        const int nHT = (sh.H + HN - 1) / HN;
        if (nHT > num_cus || nHT > 256) continue;
        // a tile's rows are addressed with 32-bit offsets
        if ((std::min(BM, sh.B) * ldmax + std::max(Kw, Kd)) * (long)es > 0x7fffffffL) continue;
        const int nBT = (sh.B + BM - 1) / BM;
        const int bgroups = std::min(std::min(nBT, num_cus / nHT), MAX_BGROUPS);
        const int G = nHT * bgroups;
        const int wrows = fwd ? 16 * NB : HN;
        const size_t red = (size_t)NWAVE * BM * (std::max(fwd ? 16 * NB : 16, 16) + 4) * 4;
        const size_t lim = (size_t)g_lds_limit - 1024;
        if (red > lim) continue;
        size_t lds = red;
        const size_t wb = (size_t)wrows * slice_pitch(Kw, es);
        const bool w_lds = lds + wb <= lim;
        if (w_lds) lds += wb;
        const int nbn = sh.Hp ? (sh.Hp + 15) / 16 : 0;
        const size_t pb = 16u * (size_t)slice_pitch(Kd, es);
        const bool p_lds = sh.Hp && nHT >= nbn && lds + pb <= lim;
        if (p_lds) lds += pb;
        const int per = (nBT + bgroups - 1) / bgroups;
        const int rows = std::min(BM, sh.B);
        double cost = SYNC_NS + per * product_ns(rows, MB, fwd ? NB : 1, (double)Kw, es, w_lds);
        if (sh.Hp) {
            const int nper = nHT >= nbn ? nHT / nbn : 1;
            const int blocks = nHT >= nbn ? 1 : (nbn + nHT - 1) / nHT;
            cost += SYNC_NS + (double)blocks * ((per + nper - 1) / nper) * product_ns(rows, MB, 1, (double)Kd, es, p_lds);
        }
        if (!found || cost < best) {
            found = true;
            best = cost;
            *out = RecTiling{HN, BM, nHT, nBT, G, bgroups, v | (w_lds ? 256 : 0) | (p_lds ? 512 : 0), lds};
        }
    }
    return found;
}

bool plan_forward(DType t, const RecShape &sh, int num_cus, RecTiling *out) { return plan(true, t, sh, num_cus, out); }
bool plan_backward(DType t, const RecShape &sh, int num_cus, RecTiling *out) { return plan(false, t, sh, num_cus, out); }

namespace {

template <typename K>
hipError_t coop_launch(K kernel, int grid, size_t lds, hipStream_t s, void *argp)
{
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    void *args[] = {argp};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(kernel), dim3(grid), dim3(WGT), args,
                                      (unsigned)lds, s);
}

template <typename TI, bool PROJ>
hipError_t fwd_dispatch(int variant, int grid, size_t lds, hipStream_t s, FwdArgs *a)
{
    switch (variant & 0xff) {
    case 0: return coop_launch(lstm_fwd_kernel<TI, 1, 1, PROJ>, grid, lds, s, a);
    case 1: return coop_launch(lstm_fwd_kernel<TI, 1, 2, PROJ>, grid, lds, s, a);
    case 2: return coop_launch(lstm_fwd_kernel<TI, 1, 4, PROJ>, grid, lds, s, a);
    case 3: return coop_launch(lstm_fwd_kernel<TI, 2, 1, PROJ>, grid, lds, s, a);
    case 4: return coop_launch(lstm_fwd_kernel<TI, 2, 2, PROJ>, grid, lds, s, a);
    case 5: return coop_launch(lstm_fwd_kernel<TI, 4, 1, PROJ>, grid, lds, s, a);
    }
    return hipErrorInvalidValue;
}

template <typename TI, bool PROJ>
hipError_t bwd_dispatch(int variant, int grid, size_t lds, hipStream_t s, BwdArgs *a)
{
    switch (VAR_MB[variant & 0xff]) {
    case 1: return coop_launch(lstm_bwd_kernel<TI, 1, PROJ>, grid, lds, s, a);
    case 2: return coop_launch(lstm_bwd_kernel<TI, 2, PROJ>, grid, lds, s, a);
    case 4: return coop_launch(lstm_bwd_kernel<TI, 4, PROJ>, grid, lds, s, a);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_forward(DType t, const RecShape &sh, const RecTiling &tl, const FwdBufs &bf, hipStream_t s)
{
    device_limits();
    const size_t es = dsize(t);
    const int Hr = sh.Hp ? sh.Hp : sh.H;
    FwdArgs a;
    a.T = sh.T; a.B = sh.B; a.H = sh.H; a.Hp = sh.Hp; a.Hr = Hr; a.reverse = sh.reverse; a.ldy = sh.ldy;
    a.R = static_cast<const char *>(bf.R);
    a.P = static_cast<const char *>(bf.P);
    a.h0 = static_cast<const char *>(bf.h0);
    a.c0 = bf.c0;
    a.gates = bf.gates; a.cs = bf.cs;
    a.ms = static_cast<char *>(bf.ms);
    a.y = static_cast<char *>(bf.y);
    a.hT = static_cast<char *>(bf.hT);
    a.cT = bf.cT;
    a.sync = bf.sync;
    a.timeout = watchdog_ticks();
    a.nHT = tl.nHT; a.nBT = tl.nBT; a.bgroups = tl.bgroups;
    a.w_lds = (tl.variant >> 8) & 1;
    a.p_lds = (tl.variant >> 9) & 1;
    a.kpitch = slice_pitch(Hr, es);
    a.ppitch = slice_pitch(sh.H, es);

    hipError_t e = fill_u32(bf.sync, SYNC_WORDS, 0u, s);   // the groups' flags and the abort word
    if (e != hipSuccess) return e;
    const double G4 = 4.0 * sh.H;
    const double flops = 2.0 * sh.T * sh.B * G4 * Hr + (sh.Hp ? 2.0 * sh.T * sh.B * sh.H * sh.Hp : 0.0);
    const double bytes = (double)sh.T * sh.B * (G4 * 8.0 + sh.H * 4.0 + Hr * (double)es + (sh.Hp ? sh.H * (double)es : 0.0)) +
                         G4 * Hr * (double)es + (sh.Hp ? (double)sh.Hp * sh.H * es : 0.0);
    ProfScope ps(K_REC_FWD, s, flops, bytes);
    if (t == DType::BF16)
        return sh.Hp ? fwd_dispatch<bf16_t, true>(tl.variant, tl.G, tl.lds, s, &a)
                     : fwd_dispatch<bf16_t, false>(tl.variant, tl.G, tl.lds, s, &a);
    return sh.Hp ? fwd_dispatch<float, true>(tl.variant, tl.G, tl.lds, s, &a)
                 : fwd_dispatch<float, false>(tl.variant, tl.G, tl.lds, s, &a);
}

hipError_t launch_backward(DType t, const RecShape &sh, const RecTiling &tl, const BwdBufs &bf, hipStream_t s)
{
    device_limits();
    const size_t es = dsize(t);
    const int Hr = sh.Hp ? sh.Hp : sh.H;
    BwdArgs a;
    a.T = sh.T; a.B = sh.B; a.H = sh.H; a.Hp = sh.Hp; a.Hr = Hr; a.reverse = sh.reverse; a.ldy = sh.ldy;
    a.Rt = static_cast<const char *>(bf.Rt);
    a.Pt = static_cast<const char *>(bf.Pt);
    a.dy = static_cast<const char *>(bf.dy);
    a.dhT = static_cast<const char *>(bf.dhT);
    a.dcT = bf.dcT; a.c0 = bf.c0; a.gates = bf.gates; a.cs = bf.cs;
    a.dz = static_cast<char *>(bf.dz);
    a.dH = static_cast<char *>(bf.dH);
    a.dh0 = static_cast<char *>(bf.dh0);
    a.dc0 = bf.dc0;
    a.dcn = bf.dcn; a.dhn = bf.dhn;
    a.dbpart = bf.dbpart;
    a.sync = bf.sync;
    a.timeout = watchdog_ticks();
    a.HN = tl.HN; a.nHT = tl.nHT; a.nBT = tl.nBT; a.bgroups = tl.bgroups;
    a.w_lds = (tl.variant >> 8) & 1;
    a.p_lds = (tl.variant >> 9) & 1;
    a.kpitch = slice_pitch(sh.Hp ? sh.Hp : 4L * sh.H, es);
    a.ppitch = slice_pitch(4L * sh.H, es);

    hipError_t e = fill_u32(bf.sync, SYNC_WORDS, 0u, s);
    if (e != hipSuccess) return e;
    const double G4 = 4.0 * sh.H;
    const double flops = 2.0 * sh.T * sh.B * G4 * Hr + (sh.Hp ? 2.0 * sh.T * sh.B * sh.H * sh.Hp : 0.0);
    const double bytes = (double)sh.T * sh.B * (G4 * 4.0 + sh.H * 4.0 + G4 * (double)es + Hr * (double)es) +
                         G4 * Hr * (double)es + (sh.Hp ? (double)sh.Hp * sh.H * es : 0.0);
    ProfScope ps(K_REC_BWD, s, flops, bytes);
    if (t == DType::BF16)
        return sh.Hp ? bwd_dispatch<bf16_t, true>(tl.variant, tl.G, tl.lds, s, &a)
                     : bwd_dispatch<bf16_t, false>(tl.variant, tl.G, tl.lds, s, &a);
    return sh.Hp ? bwd_dispatch<float, true>(tl.variant, tl.G, tl.lds, s, &a)
                 : bwd_dispatch<float, false>(tl.variant, tl.G, tl.lds, s, &a);
}

// LSTM355_WATCHDOG_US (microseconds) replaces the 2 s watchdog of the
// persistent kernels' waits: a test sets it tiny to make the kernels give up
// from the host, with every wave still exiting normally.
unsigned long long watchdog_ticks()
{
    device_limits();
    if (const char *env = std::getenv("LSTM355_WATCHDOG_US")) {
        const long us = std::atol(env);
        if (us >= 0) return g_timeout_ticks / 2000000ull * (unsigned long long)us;
    }
    return g_timeout_ticks;
}

hipError_t watchdog_read_and_clear(unsigned *tripped)
{
    unsigned v = 0;
    hipError_t e = hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_watchdog_tripped), sizeof(v), 0, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    *tripped = v;
    if (v) {
        const unsigned zero = 0;
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_watchdog_tripped), &zero, sizeof(zero), 0, hipMemcpyHostToDevice);
    }
    return e;
}

}  // namespace lstm355
