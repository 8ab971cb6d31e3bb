// Matrix-core kernels for Y = A * Omega(seed) with a wide sketch on gfx950.
//
// FP32 A (k > 8).  The product is a dense contraction (2k flops per A element).
// k = 9 .. 16: v_mfma_f32_16x16x4f32 (mfma_tile_f32).  k > 16: the FP16 matrix cores
// with both operands split into FP16 terms (sk_split.hpp: four v_mfma_f32_16x16x32_f16
// per 32 contraction columns, FP32 sums), whose error against FP64 is below that of an
// FP32 chain on dense data; what the terms cannot hold goes to f32_sums.
//
// Tile of one workgroup (64 W threads = W waves): 16 TM W rows of A x a strip of
// kMfmaStrip contraction columns x BN = 16*NT sketch columns.  Each wave owns
// TM row tiles of 16 rows x NT N-tiles, i.e. TM*NT accumulator tiles of
// Y^T (Omega is the A operand, A the B operand, so a lane's accumulators belong
// to one row of each row tile and the row's scale is the lane's own).
//
// Contraction in chunks of KC = 32 columns, one MFMA step each:
//   * A goes straight from HBM into the operand layout: lane (g, i) (g = lane/16,
//     i = lane%16) loads the 8 contiguous floats A[row i][kc + 8 g ...] of each
//     row tile as two back-to-back 16-byte loads, so each 128-byte line of a row is
//     requested at once, and splits them in registers.  Plain (temporal) loads:
//     the lines of a row are shared by the four lanes of a row.
//   * Omega's three terms for the chunk sit in one half of a double-buffered LDS
//     tile, laid out [column][b0 | b1 | b2], so that lane (g, j) reads the 8
//     contraction columns 8g .. 8g + 7 of column j as 16-byte operands.
//   * The next chunk's Omega is generated (or copied from the call's packed Omega)
//     and split while this chunk's MFMAs run; one LDS-only barrier per chunk.
// Strip partials are FP32 in [S][m][k]; the FP64 strip sum is the shared
// reduction kernel.  The order of every sum depends only on the strip
// boundaries, so results are layout independent and reproducible.
#include <algorithm>
#include <type_traits>

#include "sk_device.hpp"
#include "sk_internal.hpp"
#include "sk_split.hpp"

#pragma clang fp contract(off)

namespace sk {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

constexpr int kTM = 4;                  // M-tiles (16 rows) per wave
constexpr int kWaves = 8;               // waves per workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kBM = kWaves * kTM * 16;  // rows per workgroup
static_assert(kBM == kMfmaRows, "tile rows");
// With 8 N-tiles the raw A values are single-buffered (the accumulators take 128
// registers): they are split before a chunk's 128 MFMAs, which cover the next
// chunk's load.
constexpr bool single_a(int nt, int tm = kTM) { return nt >= 8 && tm >= kTM; }
// Chunks of Omega generated per barrier by a tile of W waves x 16 TM rows (one or two
// N-tiles): one in the 512-row tile, where the other waves' MFMAs cover a chunk's few
// Philox quads; as many as give every thread a quad in the smaller tiles, which run a
// workgroup or less per compute unit and wait for each chunk.
constexpr int tile_group(int nt, int w, int tm) {
    return tm >= kTM || nt > 2 || 64 * w < 256 * nt ? 1 : 64 * w / (128 * nt);
}

struct MArgs {
    int64_t m;
    int64_t k;
    int64_t ldy;
    int64_t ldo;
    const float* omega;
    void* Y;
    float* partials;
    uint32_t key0, key1;
    uint32_t col0;
    int dist;
    int P;
    int S_total;
    int y_f64;
    int beta;
    const uint16_t* opack;    // low-precision path: packed Omega, hi plane
    const uint16_t* opack_lo; // and lo plane
    int64_t kpad;             // sketch columns per packed chunk (k rounded up to the N-tile)
    int64_t nrt;              // row tiles
    int nblk;                 // sketch-column blocks
    const float* fpack;       // FP32 path with 4+ N-tiles: the call's packed Omega
    BlockDesc blk[kMaxBlocks];
};

// Tile of this workgroup in a one-dimensional grid of 8 * ceil(T / 8)
// workgroups over T = nblk * S_total * nrt tiles.
// XCD: workgroups are handed to the 8 XCDs
// round-robin, so XCD x runs ids x, x + 8, ...; mapping them to the contiguous
// tile range [x * T8, (x + 1) * T8), ordered sketch-column block fastest, then
// strip, then row tile, makes each XCD read whole rows of A (every strip of a
// row tile at once) and keeps the column blocks of one (strip, row tile) in
// one L2.  Measured on 32768^2 FP8 at k = 64: 290 us against 371 with the
// strip index fastest across XCDs.
// The FP32 kernel with split operands gains as well: k = 64 on 65536 x 16384 850 us
// against 876, k = 256 on 32768^2 (two column blocks) 2.23 ms against 2.43.
// Otherwise (FP32 kernel with one N-tile, the same either way): the id is the
// tile, strip fastest, then row tile, then column block.
// Returns false for the padding ids past T.
struct TileId {
    int strip;
    int64_t rtile;
    int nb;
};
template <bool XCD>
__device__ __forceinline__ bool mfma_tile_id(const MArgs& a, TileId& id) {
    const int64_t T = (int64_t)a.nblk * a.S_total * a.nrt;
    const int64_t v = blockIdx.x;
    if constexpr (XCD) {
        const int64_t T8 = (T + 7) / 8;
        const int64_t t = (v % 8) * T8 + v / 8;
        if (t >= T) return false;
        id.nb = (int)(t % a.nblk);
        const int64_t r = t / a.nblk;
        id.strip = (int)(r % a.S_total);
        id.rtile = r / a.S_total;
    } else {
        if (v >= T) return false;
        id.strip = (int)(v % a.S_total);
        const int64_t r = v / a.S_total;
        id.rtile = r % a.nrt;
        id.nb = (int)(r / a.nrt);
    }
    return true;
}

dim3 mfma_grid(const MArgs& a) {
    const int64_t T = (int64_t)a.nblk * a.S_total * a.nrt;
    return dim3((unsigned)(8 * ((T + 7) / 8)));
}

__device__ __forceinline__ void lds_barrier_m() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One tile: rows [block_row, block_row + 512) of a block, one strip of its
// columns, sketch columns [n_base, n_base + 16*NT).
struct MTile {
    const unsigned char* A;   // the block's A
    int64_t lda, n, row0;     // the block's ld, width, first Omega row
    const float* scales;
    int64_t m, k;
    int64_t col_begin;        // first column of the strip inside the block
    int64_t block_row;        // first row of the workgroup (before the wave offset)
    int n_base;
    uint32_t key0, key1, col0;
    int dist;                 // Omega's distribution (0 normal, 1 uniform, 2 Rademacher)
    const float* omega;
    int64_t ldo;
    void* Y;
    int64_t ldy;
    int y_f64, beta;
    float* partials;
    int64_t strip;            // strip index in the partial array
    bool single;
    const uint16_t* opack;    // packed Omega of the call (low-precision path), hi plane
    const uint16_t* opack_lo; // and lo plane
    int64_t kpad;
    const float* fpack;       // packed Omega of the call (FP32 path), or nullptr
};

// Arguments of the kernels that form a call's Omega once, before the product
// (k_f32_pack: one FP32 plane at hi; k_lp_pack: BF16 hi and lo planes).
struct PackArgs {
    void* hi;
    void* lo;
    int64_t k, kpad;
    uint32_t key0, key1, col0;
    int dist;
    const float* omega;       // stored Omega (n x k, ldo), or nullptr: generated
    int64_t ldo;
    int P;
    BlockDesc blk[kMaxBlocks];
};

// Write a wave's accumulators: lane (g, j) holds rows 4g..4g+3 and column j of
// each 16 x 16 tile.  The per-128-row scale (FP8 storage) is applied to each
// strip partial; a single-strip call writes Y directly (old Y added in FP64).
template <int NT, int TM = kTM>
__device__ __forceinline__ void store_tile(const MTile& t, const v4f (&acc)[TM][NT],
                                           int64_t row_base, int kb, int g, int i16) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int cn = nt * 16 + i16;
            if (cn >= kb) continue;
            const int64_t col = t.n_base + cn;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int64_t r = row_base + tm * 16 + 4 * g + rr;
                if (r >= t.m) continue;
                float v = acc[tm][nt][rr];
                if (t.scales) v *= t.scales[r >> 7];
                if (t.single) {
                    double y = (double)v;
                    if (t.y_f64) {
                        double* Yp = static_cast<double*>(t.Y) + r * t.ldy + col;
                        if (t.beta) y += *Yp;
                        *Yp = y;
                    } else {
                        float* Yp = static_cast<float*>(t.Y) + r * t.ldy + col;
                        if (t.beta) y += (double)*Yp;
                        *Yp = (float)y;
                    }
                } else {
                    t.partials[(t.strip * t.m + r) * t.k + col] = v;
                }
            }
        }
    }
}

// Columns past k of an LDS ring of `slots` chunks are zeroed once: generation never
// writes them.
template <int BN, int TH>
__device__ __forceinline__ void omega_zero_pad(_Float16 (*om)[BN][kSplitRow], int slots, int kb) {
    for (int it = threadIdx.x; it < slots * BN * (kSplitRow / 8); it += TH) {
        const int n = (it / (kSplitRow / 8)) % BN;
        if (n >= kb) reinterpret_cast<v4u*>(&om[0][0][0])[it] = v4u{0u, 0u, 0u, 0u};
    }
}

// Chunks c0 .. c0 + G - 1 (those below nchunks) of the tile's strip, sketch columns
// n_base .. n_base + kb - 1, split into LDS slots slot0 .. (slot0 + G - 1); zeros past
// the strip's end.  Generated from the seed, or read from a stored Omega.  With few sketch
// columns one chunk has too few Philox quads to occupy the workgroup, G of them do.  A
// chunk's first Omega row is aligned as the strip's (chunk widths are multiples of 4), so
// every chunk has the same quad count.
template <int BN, int TH, int G, bool GEN>
__device__ __forceinline__ void omega_group(const MTile& t, _Float16 (*om)[BN][kSplitRow],
                                            int slot0, int c0, int nchunks, int w, int kb) {
    constexpr int KC = kSplitKC;
    const int cnt = min(G, nchunks - c0);
    const float sc = __builtin_ldexpf(1.0f, kOmegaExp);
    if constexpr (GEN) {
        const int64_t gb = t.row0 + t.col_begin;                     // Omega row of strip column 0
        const int nq = (int)(((gb + KC - 1) >> 2) - (gb >> 2) + 1);   // KC/4, or one more if unaligned
        const int per = nq * kb;
        for (int it = threadIdx.x; it < cnt * per; it += TH) {
            const int ci = it / per;
            const int r = it - ci * per;
            const int qi = r / kb;
            const int n = r - qi * kb;
            const int c = c0 + ci;
            const int64_t g0 = gb + (int64_t)c * KC;
            const int kvalid = min(KC, w - c * KC);
            const int64_t q = (g0 >> 2) + qi;
            const float4 z = omega4_dist((uint64_t)q, t.col0 + (uint32_t)(t.n_base + n), t.key0,
                                         t.key1, t.dist);
            const int kl0 = (int)(4 * q - g0);
            _Float16* dst = om[slot0 + ci][n];
            if (kl0 >= 0 && (kl0 & 3) == 0 && kl0 + 3 < kvalid) {
                split_store4(dst, kl0, f32x4{z.x, z.y, z.z, z.w}, sc);
            } else {
                const float zz[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int kl = kl0 + u;
                    if (kl >= 0 && kl < KC) split_store1(dst, kl, (kl < kvalid) ? zz[u] : 0.0f, sc);
                }
            }
        }
    } else {
        for (int it = threadIdx.x; it < cnt * KC * kb; it += TH) {
            const int ci = it / (KC * kb);
            const int r = it - ci * (KC * kb);
            const int kl = r / kb;
            const int n = r - kl * kb;
            const int c = c0 + ci;
            float z = 0.0f;
            if (c * KC + kl < w)
                z = t.omega[(t.col_begin + (int64_t)c * KC + kl) * t.ldo + t.n_base + n];
            split_store1(om[slot0 + ci][n], kl, z, sc);
        }
    }
}

// ---- Omega of a whole call for the FP32 tiles (four or more N-tiles) ---------
// As for the low-precision route: every 512-row tile of a strip multiplies the
// same Omega chunks, so the call forms them once.  One FP32 plane, chunk
// gc = strip * (kMfmaStrip / 32) + c, then sketch column n in [0, kpad), then
// contraction column kl in [0, 32): element (gc * kpad + n) * 32 + kl; the
// values (zeros past the strip's end and for n >= k) are those omega_group
// writes into LDS, so the sums are the same bit for bit.
constexpr int kF32PackRows = 16;   // sketch columns per packing workgroup
constexpr bool mfma_packed(int nt) { return nt >= 4; }

// grid (chunks of all strips / kF32PackChunks, ceil(kpad / 16)); 256 threads.
// A workgroup forms kF32PackChunks consecutive chunks of one strip (a strip is
// 64 chunks), so that its threads have Philox quads enough to keep busy.
constexpr int kF32PackChunks = 4;

template <bool GEN>
__global__ __launch_bounds__(256) void k_f32_pack(const PackArgs a) {
    constexpr int KC = kSplitKC;
    constexpr int CPS = kMfmaStrip / KC;
    constexpr int G = kF32PackChunks;
    static_assert(CPS % G == 0, "groups of chunks inside a strip");
    __shared__ __attribute__((aligned(16))) float sh[G][kF32PackRows][KC + 4];
    const int tid = threadIdx.x;
    const int64_t gc0 = (int64_t)blockIdx.x * G;          // first chunk of the group
    const int64_t strip = gc0 / CPS;
    const int c0 = (int)(gc0 - strip * CPS);
    int b = 0;
    int64_t sib = strip;
    for (; b < a.P; ++b) {
        const int64_t sb = (a.blk[b].n + kMfmaStrip - 1) / kMfmaStrip;
        if (sib < sb) break;
        sib -= sb;
    }
    const int64_t col_begin = sib * kMfmaStrip;
    const int w = (int)min<int64_t>(kMfmaStrip, a.blk[b].n - col_begin);
    const int nc = min(G, (w - c0 * KC + KC - 1) / KC);   // chunks of the group inside the strip
    if (nc <= 0) return;                                  // past the strip's end: never read
    const int nb0 = blockIdx.y * kF32PackRows;
    const int kb = (int)min<int64_t>(kF32PackRows, a.k - nb0);   // <= 0: all zero
    for (int it = tid; it < G * kF32PackRows * (KC + 4); it += 256) (&sh[0][0][0])[it] = 0.0f;
    __syncthreads();
    if constexpr (GEN) {
        // every chunk starts at the same offset within a Philox quad (KC is a multiple of 4)
        const int64_t gs = a.blk[b].row0 + col_begin + (int64_t)c0 * KC;
        const int nq = (int)(((gs + KC - 1) >> 2) - (gs >> 2) + 1);
        const int per = kb > 0 ? nq * kb : 0;
        for (int it = tid; it < nc * per; it += 256) {
            const int ci = it / per;
            const int r = it - ci * per;
            const int qi = r / kb;
            const int n = r - qi * kb;
            const int64_t g0 = gs + (int64_t)ci * KC;
            const int kvalid = min(KC, w - (c0 + ci) * KC);
            const int64_t q_lo = g0 >> 2;
            const float4 z = omega4_dist((uint64_t)(q_lo + qi), a.col0 + (uint32_t)(nb0 + n),
                                         a.key0, a.key1, a.dist);
            const int kl0 = (int)(4 * (q_lo + qi) - g0);
            const float zz[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int kl = kl0 + u;
                if (kl >= 0 && kl < kvalid) sh[ci][n][kl] = zz[u];
            }
        }
    } else {
        const int per = kb > 0 ? KC * kb : 0;
        for (int it = tid; it < nc * per; it += 256) {
            const int ci = it / per;
            const int r = it - ci * per;
            const int kl = r / kb;
            const int n = r - kl * kb;
            if (kl < min(KC, w - (c0 + ci) * KC))
                sh[ci][n][kl] = a.omega[(col_begin + (int64_t)(c0 + ci) * KC + kl) * a.ldo + nb0 + n];
        }
    }
    __syncthreads();
    const int rows = (int)min<int64_t>(kF32PackRows, a.kpad - nb0);
    const int ppc = rows * (KC / 4);                      // 16-byte pieces per chunk
    float* out = static_cast<float*>(a.hi);
    for (int it = tid; it < nc * ppc; it += 256) {
        const int ci = it / ppc;
        const int pc = it - ci * ppc;
        const int n = pc / (KC / 4);
        const int kl4 = (pc - n * (KC / 4)) * 4;
        *reinterpret_cast<v4f*>(out + (((gc0 + ci) * a.kpad + nb0 + n) * KC + kl4)) =
            *reinterpret_cast<const v4f*>(&sh[ci][n][kl4]);
    }
}

// Write v as the strip sum (row, col) of a tile: scaled, to the partials, or to Y of a
// single-strip call (old Y added in FP64).
struct TileOut {
    const float* scales;
    float* partials;          // strip's first partial, or nullptr: single strip
    void* Y;
    int64_t k, ldy;
    int y_trans, y_f64, beta;
    // runs of four sketch columns lie 16-byte aligned and are only stored
    __device__ __forceinline__ bool vec() const {
        return !scales && (partials ? (k & 3) == 0
                                    : !(y_trans || y_f64 || beta) && (ldy & 3) == 0 &&
                                          ((uintptr_t)Y & 15) == 0);
    }
};
__device__ __forceinline__ void emit(const TileOut& o, int64_t row, int64_t col, float v) {
    if (o.scales) v *= o.scales[row >> 7];
    if (o.partials) {
        o.partials[row * o.k + col] = v;
        return;
    }
    const int64_t off = o.y_trans ? col * o.ldy + row : row * o.ldy + col;
    double y = (double)v;
    if (o.y_f64) {
        double* Yp = static_cast<double*>(o.Y) + off;
        if (o.beta) y += *Yp;
        *Yp = y;
    } else {
        float* Yp = static_cast<float*>(o.Y) + off;
        if (o.beta) y += (double)*Yp;
        *Yp = (float)y;
    }
}

// Sketch columns col .. col + 3 (col a multiple of 4) of a row, those below `end` that
// `skip` leaves.
__device__ __forceinline__ void emit4(const TileOut& o, bool vec, int64_t row, int64_t col,
                                      int64_t end, const v4f u, const bool (&skip)[4]) {
    if (vec && col + 3 < end && !(skip[0] || skip[1] || skip[2] || skip[3])) {
        float* p = o.partials ? o.partials + row * o.k : static_cast<float*>(o.Y) + row * o.ldy;
        *reinterpret_cast<v4f*>(p + col) = u;
        return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (col + r < end && !skip[r]) emit(o, row, col + r, u[r]);
}

// The lane's accumulator of one 16 x 16 tile of Y^T, of a row with scale s.  Columns that
// f32_sums evaluates (f32col, of a stored Omega) are left to it: with one strip and beta = 1
// a second store would add to the first.
__device__ __forceinline__ void emit_split(const TileOut& o, bool vec, int64_t row, int64_t col,
                                           int64_t end, const v4f v, float s, const int* f32col) {
    v4f u;
    bool skip[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        u[r] = unscale(v[r], s);
        skip[r] = f32col && f32col[r];
    }
    emit4(o, vec, row, col, end, u, skip);
}

constexpr int kF32Row = kSplitKC + 4;   // floats per LDS column of an FP32 chunk
template <int TH, bool GEN>
__device__ __forceinline__ void omega_chunk_f32(const MTile& t, float (*om)[kF32Row], int c, int w,
                                                int kb, int first) {
    // thread `first` takes the first item
    const int start = (int)threadIdx.x >= first ? (int)threadIdx.x - first
                                                : (int)threadIdx.x - first + TH;
    constexpr int KC = kSplitKC;
    const int kvalid = min(KC, w - c * KC);
    if constexpr (GEN) {
        const int64_t g0 = t.row0 + t.col_begin + (int64_t)c * KC;   // global Omega row of local 0
        const int64_t q_lo = g0 >> 2;
        const int nq = (int)(((g0 + KC - 1) >> 2) - q_lo + 1);        // KC/4, or one more if unaligned
        for (int it = start; it < nq * kb; it += TH) {
            const int qi = it / kb;
            const int n = it - qi * kb;
            const float4 z = omega4_dist((uint64_t)(q_lo + qi), t.col0 + (uint32_t)(t.n_base + n),
                                         t.key0, t.key1, t.dist);
            const int kl0 = (int)(4 * (q_lo + qi) - g0);
            if (kl0 >= 0 && (kl0 & 3) == 0 && kl0 + 3 < kvalid) {
                *reinterpret_cast<float4*>(&om[n][kl0]) = z;
            } else {
                const float zz[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int kl = kl0 + u;
                    if (kl >= 0 && kl < KC) om[n][kl] = (kl < kvalid) ? zz[u] : 0.0f;
                }
            }
        }
    } else {
        for (int it = start; it < KC * kb; it += TH) {
            const int kl = it / kb;
            const int n = it - kl * kb;
            om[n][kl] = (kl < kvalid)
                            ? t.omega[(t.col_begin + (int64_t)c * KC + kl) * t.ldo + t.n_base + n]
                            : 0.0f;
        }
    }
}

// The strip sums of a tile's rows with row_f32[tm] (the lane's row of its row tile tm) and
// columns with f32col (nullptr: none), or all of them, with the FP32 matrix instruction: what
// the FP16 terms cannot hold (a row of A with an infinity, whose terms would meet zeros and
// the other sign, and the columns of stored_columns), and strips narrower than a chunk, whose
// few FP32 roundings are less than what the terms leave out (1 to 15 columns of N(0,1):
// 2.5e-8 to 7e-8 against 7e-8).
// Every wave of the workgroup takes part; `rows`: this one has rows.  load(x, c) gives chunk
// c of A as ALoads does, row_of(tm) the lane's row of tile tm.  Omega's chunks go through LDS
// (`om`, two halves of 16 NT columns) as in mfma_tile; the product of 32 columns is eight
// MFMAs in the order of the contraction index 8 g + e, so that the sums depend neither on the
// tile nor on A's storage order.
template <int NT, int TM, int TH, bool GEN, bool PK, typename Load, typename RowOf>
__device__ __forceinline__ void f32_sums(const MTile& t, const TileOut& o, float* om_lds, int w, int kb,
                                         bool rows, Load load, RowOf row_of, bool all,
                                         const bool (&row_f32)[TM], const int* f32col) {
    constexpr int KC = kSplitKC, BN = 16 * NT;
    // copied Omega: 16-byte pieces of the packed plane, or single values of a stored one (row
    // by row), OPT per thread; values past the strip's end or k columns are zeros
    constexpr int PPL = PK ? BN * KC / 4 : BN * KC, OPT = (PPL + TH - 1) / TH;
    using Piece = std::conditional_t<PK, v4f, float>;
    constexpr bool COPY = PK || !GEN;
    float (*om)[BN][kF32Row] = reinterpret_cast<float (*)[BN][kF32Row]>(om_lds);
    const int tid = threadIdx.x, g = (tid & 63) >> 4, i16 = tid & 15;
    const int nchunks = (w + KC - 1) / KC;
    auto om_load = [&](Piece* r, int c) {
        if constexpr (PK) {
            const int64_t gc = t.strip * (kMfmaStrip / KC) + min(c, nchunks - 1);
            const float* p = t.fpack + (gc * t.kpad + t.n_base) * KC;
#pragma unroll
            for (int j = 0; j < OPT; ++j)
                r[j] = *reinterpret_cast<const v4f*>(p + 4 * min(tid + j * TH, PPL - 1));
        } else if constexpr (COPY) {
#pragma unroll
            for (int j = 0; j < OPT; ++j) {
                const int q = tid + j * TH, kl = c * KC + q / BN, n = q % BN;
                r[j] = t.omega[(t.col_begin + min(kl, w - 1)) * t.ldo + t.n_base + min(n, kb - 1)];
                r[j] = kl < w && n < kb ? r[j] : 0.0f;
            }
        }
    };
    auto om_store = [&](const Piece* r, int c) {
#pragma unroll
        for (int j = 0; j < OPT; ++j) {
            const int q = min(tid + j * TH, PPL - 1);
            if constexpr (PK) *reinterpret_cast<v4f*>(&om[c & 1][q / (KC / 4)][(q % (KC / 4)) * 4]) = r[j];
            else om[c & 1][q % BN][q / BN] = r[j];
        }
    };
    v4f acc[TM][NT];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[tm][nt] = v4f{0.f, 0.f, 0.f, 0.f};
    float x0[TM][8], x1[TM][8];
    static_assert(PK || PPL % TH == 0, "whole values per thread");
    Piece r[COPY ? OPT : 1];
    if constexpr (COPY) {
        om_load(r, 0);
        if (rows) load(x0, 0);
        om_store(r, 0);
        om_load(r, 1);
        if (rows) load(x1, min(1, nchunks - 1));
    } else {
        // (generated: rows with an infinity, or a strip of one chunk: no load without a use)
        if (rows) load(x0, 0);
        if (rows && nchunks > 1) load(x1, 1);
        for (int it = tid; it < 2 * BN * kF32Row; it += TH)
            if ((it / kF32Row) % BN >= kb) (&om[0][0][0])[it] = 0.0f;
        omega_chunk_f32<TH, true>(t, om[0], 0, w, kb, 0);
    }
    lds_barrier_m();
    auto step = [&](float (&x)[TM][8], int c) {
        if constexpr (COPY) {
            om_store(r, c + 1);
            om_load(r, c + 2);
        } else if (c + 1 < nchunks) {
            omega_chunk_f32<TH, true>(t, om[(c + 1) & 1], c + 1, w, kb, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (rows) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    const v4f z = *reinterpret_cast<const v4f*>(&om[c & 1][nt * 16 + i16][8 * g + 4 * v]);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int tm = 0; tm < TM; ++tm)
                            acc[tm][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[e], x[tm][4 * v + e],
                                                                               acc[tm][nt], 0, 0, 0);
                }
            if (COPY || c + 2 < nchunks) load(x, min(c + 2, nchunks - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier_m();
    };
#pragma unroll 1
    for (int c = 0; c < nchunks; c += 2) {
        step(x0, c);
        if (c + 1 < nchunks) step(x1, c + 1);
    }
    if (!rows) return;
    const bool vec = o.vec();
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int64_t row = row_of(tm);
        if (row >= t.m) continue;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int c = nt * 16 + 4 * g;
            bool skip[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) skip[q] = !(all || row_f32[tm] || (f32col && f32col[c + q]));
            emit4(o, vec, row, t.n_base + c, t.n_base + kb, acc[tm][nt], skip);
        }
    }
}

// Which columns of a stored Omega the FP16 terms would not serve in the tile's strip.  The
// terms of a row of A hold its entries down to 2^-35 of the largest and those of Omega an
// entry to within 2^-49; under entries like N(0,1) ones that stays below an FP32 sum's
// rounding, but zeros (sparse or selecting columns) or a wide range can bring out a row's
// small entries alone.  So the strip's w >= 32 entries of a column have to be such as could
// have been generated: no zero, none above 6 in modulus (generated ones reach 5.77), at most
// 8 + w/64 below 2^-10 and 3 below 2^-25.  Generated columns exceed these counts with a
// probability under 1e-18 each: a stored copy multiplies with the same bits.
// f32col[n] = kOther for another column: then the tile multiplies all of its columns with
// f32_sums (65536 x 16384 at k = 64: 1278 us, and 1212 with the FP32 instruction alone, before
// the terms; 940 to 960 with the terms); kNonFinite for one with an infinity or NaN, which
// goes there alone.
constexpr int kOther = 1, kNonFinite = 2;
template <int BN, int TH, bool PK>
__device__ __forceinline__ void stored_columns(const MTile& t, int* f32col, int w, int kb) {
    // counts in one word: entries below 2^-10, below 2^-25, never generated, non-finite
    constexpr int kSmall = 1, kTiny = 1 << 12, kNever = 1 << 24, kInf = 1 << 25;
    auto grade = [=](int b) {
        if (b >= 0x7F800000) return kInf;
        if (b == 0 || b > __float_as_int(6.0f)) return kNever;
        return b < __float_as_int(0x1p-25f) ? kSmall + kTiny : b < __float_as_int(0x1p-10f) ? kSmall : 0;
    };
    auto add = [=](int sum, int q) { return q >= kNever ? sum | q : sum + q; };
    for (int n = threadIdx.x; n < BN; n += TH) f32col[n] = 0;
    __syncthreads();
    auto count = [=](int n, int sum) {
        const int mark = sum & (kNever | kInf);
        if (mark & ~f32col[n]) atomicOr(&f32col[n], mark);     // a sparse column has many
        if (sum & (kNever - 1)) atomicAdd(&f32col[n], sum & (kNever - 1));
    };
    // one such column sends the whole tile to f32_sums: no need to look further, and which
    // column is marked makes no difference
    auto settled = [=](int sum) {
        if (sum & kNever) atomicOr(&f32col[0], kNever);
        return (*(volatile int*)f32col & kNever) != 0;
    };
    if constexpr (PK) {
        // a chunk's BN columns are one run of the packed plane: thread tid's V pieces of
        // four values lie in the same columns and rows of every chunk
        constexpr int kPieces = kSplitKC / 4;
        constexpr int V = BN * kPieces / TH;
        static_assert(V * TH == BN * kPieces, "whole pieces per thread");
        constexpr int CPS = kMfmaStrip / kSplitKC;
        int sum[V], wv[V];                     // wv: the plane holds zeros past kb columns
#pragma unroll
        for (int v = 0; v < V; ++v) {
            sum[v] = 0;
            wv[v] = (threadIdx.x + v * TH) / kPieces < kb ? w : 0;
        }
        const int nch = (w + kSplitKC - 1) / kSplitKC;
        const int row = 4 * (threadIdx.x % kPieces);       // of the pieces, within a chunk
#pragma unroll 8
        for (int c = 0; c < nch; ++c) {
            const float* p = t.fpack + ((t.strip * CPS + c) * t.kpad + t.n_base) * kSplitKC;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const v4f x = *reinterpret_cast<const v4f*>(p + 4 * (threadIdx.x + v * TH));
                int b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) b[u] = __float_as_int(x[u]) & 0x7FFFFFFF;
                if (max(max(b[0], b[1]), max(b[2], b[3])) > __float_as_int(6.0f) ||
                    min(min(b[0], b[1]), min(b[2], b[3])) < __float_as_int(0x1p-10f)) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (c * kSplitKC + row + u < wv[v]) sum[v] = add(sum[v], grade(b[u]));
                }
            }
            if (c % 8 == 7 && settled(sum[0])) break;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) count((threadIdx.x + v * TH) / kPieces, sum[v]);
    } else {
        // sixteen loads in flight per thread
        constexpr int L = 16;
        const int total = w * kb;
        for (int it0 = threadIdx.x; it0 < total; it0 += L * TH) {
            float x[L];
            int n[L];
#pragma unroll
            for (int u = 0; u < L; ++u) {
                const int it = min(it0 + u * TH, total - 1);
                const int j = it / kb;
                n[u] = it - j * kb;
                x[u] = t.omega[(t.col_begin + j) * t.ldo + t.n_base + n[u]];
            }
#pragma unroll
            for (int u = 0; u < L; ++u)
                if (it0 + u * TH < total) count(n[u], grade(__float_as_int(x[u]) & 0x7FFFFFFF));
            if (settled(0)) break;
        }
    }
    __syncthreads();
    for (int n = threadIdx.x; n < kb; n += TH) {
        const int q = f32col[n];
        const bool many = q % kNever / kTiny > 3 || q % kTiny > 8 + w / 64;
        f32col[n] = q & kNever ? kOther : q & kInf ? kNonFinite : many ? kOther : 0;
    }
    __syncthreads();
}

// A operand loads of a wave: chunk c of rows row_base .. row_base + 16 TM - 1, lane (g, i) the 8
// floats at columns 8 g .. of row (tm, i).
// FULL: every block of the launch has at least one whole chunk of columns.  Then every
// lane issues the same loads every chunk, unconditionally (a load past the strip's
// whole chunks re-reads the last of them, or the one before the strip), and the
// compiler waits for the chunk being multiplied alone; with a per-lane tail path in
// the loop it waits for every load in flight, including the next chunk's, which
// undoes the double buffering.  A ragged last chunk is loaded behind a wave-uniform
// branch that waits for its own loads.  Narrower blocks take the per-lane path.
template <int TM, bool FULL>
struct ALoads {
    const unsigned char* arow[TM];
    int g, w;
    __device__ __forceinline__ ALoads(const MTile& t, int64_t row_base, int g_, int i16, int w_)
        : g(g_), w(w_) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int64_t r = min<int64_t>(row_base + tm * 16 + i16, t.m - 1);
            arow[tm] = t.A + r * (t.lda * 4) + (t.col_begin + 8 * g) * 4;
        }
    }
    __device__ __forceinline__ void load(v4f (*a)[2], int c) const {
        constexpr int KC = kSplitKC;
        const int nfull = w / KC;
        if constexpr (FULL) {
            const int cc = c < nfull ? c : nfull - 1;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const unsigned char* p = arow[tm] + (int64_t)cc * KC * 4;
#pragma unroll
                for (int v = 0; v < 2; ++v) a[tm][v] = *reinterpret_cast<const v4f*>(p + 16 * v);
            }
            if (c != nfull) return;
            asm volatile("" : "+s"(c));    // the tail's addresses are formed here, not kept
        }
        const int kl = c * KC + 8 * g;                      // strip column of component 0
        if (c * KC >= w) return;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const unsigned char* p = arow[tm] + (int64_t)c * KC * 4;
            if (kl + 7 < w) {
#pragma unroll
                for (int v = 0; v < 2; ++v) a[tm][v] = *reinterpret_cast<const v4f*>(p + 16 * v);
            } else {
                const float* pf = reinterpret_cast<const float*>(p);
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    v4f x = {0.f, 0.f, 0.f, 0.f};
                    for (int e = 0; e < 4; ++e)
                        if (kl + 4 * v + e < w) x[e] = pf[4 * v + e];
                    a[tm][v] = x;
                }
            }
        }
        if constexpr (FULL) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) asm volatile("" : "+v"(a[tm][0]), "+v"(a[tm][1]));
        }
    }
};

// k <= 16 (one N-tile): v_mfma_f32_16x16x4f32.  Reading A bounds these sketches, and
// this tile's few registers (no terms to hold) keep more loads in flight: 65536 x 16384 at
// k = 16 takes 767 us here and 800 us with split operands.  Same tile, loads and barriers as
// mfma_tile; A is the A operand, 8 MFMAs per chunk and row tile: component s of 16-byte load
// v is contraction index g of MFMA 4v + s.  FULL as for mfma_tile.
template <int G>
struct F32Lds {
    float om[2 * G][16][kF32Row];
};

template <int W, int TM, bool GEN, bool FULL>
__device__ __forceinline__ void mfma_tile_f32(const MTile& t, F32Lds<tile_group(1, W, TM)>& L) {
    constexpr int TH = 64 * W;
    constexpr int G = tile_group(1, W, TM);
    constexpr int KC = kSplitKC;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int g = lane >> 4;
    const int i16 = lane & 15;

    const int w = (int)min<int64_t>(kMfmaStrip, t.n - t.col_begin);
    const int nchunks = (w + KC - 1) / KC;
    const int64_t row_base = t.block_row + wave * (TM * 16);
    const int kb = (int)min<int64_t>(16, t.k - t.n_base);
    const ALoads<TM, FULL> A(t, row_base, g, i16, w);

    // columns past k of every slot are zeroed once: generation never writes them
    for (int it = threadIdx.x; it < 2 * G * 16 * kF32Row; it += TH)
        if ((it / kF32Row) % 16 >= kb) (&L.om[0][0][0])[it] = 0.0f;
    // chunks c .. c + G - 1, one call each: their quads go to different threads
    auto make_group = [&](int c) {
#pragma unroll
        for (int u = 0; u < G; ++u)
            if (c + u < nchunks)
                omega_chunk_f32<TH, GEN>(t, L.om[(c + u) & (2 * G - 1)], c + u, w, kb, u * (TH / G));
    };

    v4f acc[TM][1];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) acc[tm][0] = v4f{0.f, 0.f, 0.f, 0.f};
    v4f a0[TM][2], a1[TM][2];
    A.load(a0, 0);
    A.load(a1, 1);
    make_group(0);
    lds_barrier_m();
    auto step = [&](v4f (*a)[2], int c) {
        if (c % G == 0) make_group(c + G);
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const v4f bop = *reinterpret_cast<const v4f*>(&L.om[c & (2 * G - 1)][i16][8 * g + 4 * v]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
                    acc[tm][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[tm][v][s], bop[s], acc[tm][0],
                                                                      0, 0, 0);
        }
        A.load(a, c + 2);
        if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
        if (c % G == G - 1) lds_barrier_m();
    };
    for (int c = 0; c < nchunks; c += 2) {
        step(a0, c);
        if (c + 1 < nchunks) step(a1, c + 1);
    }
    store_tile<1, TM>(t, acc, row_base, kb, g, i16);
}

// Split operands (two or more N-tiles).
// PK: Omega chunks copied from the call's packed Omega (k_f32_pack) and split on the
// way to LDS; the copy of chunk c + 2 is issued ahead of the A loads issued after it,
// so waiting for it leaves those in flight.
template <int NT, int G>
struct SplitLds {
    union {
        _Float16 om[2 * G][16 * NT][kSplitRow];
        float f32[2][16 * NT][kF32Row];
    };
    int f32col[16 * NT];           // of a stored Omega, see stored_columns
};

template <int NT, int W, int TM, bool GEN, bool FULL = false, bool PK = false>
__device__ __forceinline__ void mfma_tile(const MTile& t, SplitLds<NT, tile_group(NT, W, TM)>& L) {
    constexpr int G = PK ? 1 : tile_group(NT, W, TM);   // chunks generated per barrier
    constexpr int BN = 16 * NT;
    constexpr int TH = 64 * W;
    constexpr int KC = kSplitKC;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4;      // contraction group of the lane (both operands)
    const int i16 = lane & 15;    // A row / sketch column within a tile
    _Float16 (*om)[BN][kSplitRow] = L.om;

    const int w = (int)min<int64_t>(kMfmaStrip, t.n - t.col_begin);
    const int nchunks = (w + KC - 1) / KC;
    const int64_t row_base = t.block_row + wave * (TM * 16);
    const int n_base = t.n_base;
    const int kb = (int)min<int64_t>(BN, t.k - n_base);
    const bool stored = (PK || !GEN) && t.omega != nullptr;   // uniform across the launch

    const ALoads<TM, FULL> A(t, row_base, g, i16, w);

    // the tile has nothing for the FP16 terms (uniform across the workgroup)
    bool f32_all = w < KC;
    if (stored && !f32_all) {
        stored_columns<BN, TH, PK>(t, L.f32col, w, kb);
        bool other = false;
        for (int n = lane; n < kb; n += 64) other = other || L.f32col[n] == kOther;
        f32_all = __any(other);                      // alike in every wave
    }

    // ---- Omega chunk -> LDS ----------------------------------------------------------
    auto make_group = [&](int c) {
        omega_group<BN, TH, G, GEN>(t, om, c & (2 * G - 1), c, nchunks, w, kb);
    };
    // packed route: 16-byte pieces of the tile's run of a chunk, OPT per thread;
    // chunk indices past the last are clamped (a re-read of valid memory whose
    // copy lands in the LDS half no step reads next)
    constexpr int PPL = BN * KC / 4;
    constexpr int OPT = (PPL + TH - 1) / TH;
    static_assert(!PK || PPL % TH == 0, "whole pieces per thread");
    auto om_load = [&](v4f* r, int c) {
        const int cc = c < nchunks ? c : nchunks - 1;
        const char* src = reinterpret_cast<const char*>(
            t.fpack + ((t.strip * (kMfmaStrip / KC) + cc) * t.kpad + n_base) * KC);
        // a scalar base and 32-bit lane offsets: a 64-bit base per lane was spilled in the
        // eight-N-tile loop, and its reload waited for the A loads in flight
#pragma unroll
        for (int j = 0; j < OPT; ++j)
            r[j] = *reinterpret_cast<const v4f*>(src + 16u * (uint32_t)(tid + j * TH));
    };
    auto om_store = [&](const v4f* r, int c) {
        const int buf = c & 1;
#pragma unroll
        for (int j = 0; j < OPT; ++j) {
            const int p = tid + j * TH;
            split_store4(om[buf][p / (KC / 4)], (p % (KC / 4)) * 4, r[j], 0x1p13f);
        }
    };

    v4f acc[TM][NT];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[tm][nt] = v4f{0.f, 0.f, 0.f, 0.f};
    float s[TM];                 // scale of row (tm, i16)
    bool inf[TM];                // the row holds an infinity
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        s[tm] = kRowStart;
        inf[tm] = false;
    }

    // chunk's raw values -> MFMA operands, rescaling rows that outgrow FP16
    h8 a0[TM], a1[TM], a0s[TM];
    auto split = [&](v4f (*a)[2]) {
        float x[TM][8], y[TM][8];
        float mx = 0.0f;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[tm][e] = a[tm][e >> 2][e & 3];
                y[tm][e] = x[tm][e] * s[tm];
            }
            mx = absmax8(y[tm], mx);
        }
        if (__builtin_expect(__any(mx > kRowLimit), 0)) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const float f = rescale_row(x[tm], s[tm], inf[tm]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[tm][nt] *= f;
#pragma unroll
                for (int e = 0; e < 8; ++e) y[tm][e] = x[tm][e] * s[tm];
            }
        }
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) split_a(y[tm], a0[tm], a1[tm], a0s[tm]);
    };

    auto compute = [&](int c) {
        const int buf = c & (2 * G - 1);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const _Float16* ob = &om[buf][nt * 16 + i16][8 * g];
            const h8 b0 = *reinterpret_cast<const h8*>(ob);
            const h8 b1 = *reinterpret_cast<const h8*>(ob + KC);
            const h8 b2 = *reinterpret_cast<const h8*>(ob + 2 * KC);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                acc[tm][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a1[tm], acc[tm][nt], 0, 0, 0);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                acc[tm][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b2, a0s[tm], acc[tm][nt], 0, 0, 0);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                acc[tm][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b1, a0s[tm], acc[tm][nt], 0, 0, 0);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                acc[tm][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a0[tm], acc[tm][nt], 0, 0, 0);
        }
    };

    if (!f32_all) {
        if constexpr (!PK) omega_zero_pad<BN, TH>(om, 2 * G, kb);
        v4f r0[TM][2], r1[TM][2];
        v4f orr[PK ? OPT : 1];
        if constexpr (PK) {
            om_load(orr, 0);
            A.load(r0, 0);
            om_store(orr, 0);
            om_load(orr, 1);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!single_a(NT, TM)) A.load(r1, 1);
        } else {
            A.load(r0, 0);
            if constexpr (!single_a(NT, TM)) A.load(r1, 1);
            make_group(0);
        }
        lds_barrier_m();

        // step c: chunk c + 1's Omega to LDS, chunk c's A split, its registers refilled,
        // chunk c's MFMAs
        auto step = [&](v4f (*r)[2], int c) {
            if constexpr (PK) {
                om_store(orr, c + 1);
                om_load(orr, c + 2);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                if (c % G == 0 && c + G < nchunks) make_group(c + G);
            }
            split(r);
            A.load(r, c + (single_a(NT, TM) ? 1 : 2));
            if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
            compute(c);
            if (c % G == G - 1) lds_barrier_m();
        };
        if constexpr (single_a(NT, TM)) {
            for (int c = 0; c < nchunks; ++c) step(r0, c);
        } else {
            for (int c = 0; c < nchunks; c += 2) {
                step(r0, c);
                if (c + 1 < nchunks) step(r1, c + 1);
            }
        }
    }

    // ---- lane (g, i) holds sketch columns 4g .. 4g + 3 of row i of each tile ------
    TileOut o;
    o.scales = t.scales;
    o.partials = t.single ? nullptr : t.partials + t.strip * t.m * t.k;
    o.Y = t.Y;
    o.k = t.k;
    o.ldy = t.ldy;
    o.y_trans = 0;
    o.y_f64 = t.y_f64;
    o.beta = t.beta;
    const bool vec = o.vec();
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int64_t row = row_base + tm * 16 + i16;
        if (f32_all || row >= t.m || inf[tm]) continue;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            emit_split(o, vec, row, n_base + nt * 16 + 4 * g, n_base + kb, acc[tm][nt], s[tm],
                       stored ? &L.f32col[nt * 16 + 4 * g] : nullptr);
    }
    // ---- rows and columns for FP32 products --------------------------------------------
    bool redo = f32_all;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) redo = redo || inf[tm];
    if (stored)
        for (int n = lane; n < kb; n += 64) redo = redo || L.f32col[n];
    if (__syncthreads_or(redo)) {
        f32_sums<NT, TM, TH, GEN, PK>(
            t, o, &L.f32[0][0][0], w, kb, true,
            [&](float (&x)[TM][8], int c) {
                v4f r[TM][2];
                A.load(r, c);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[tm][e] = r[tm][e >> 2][e & 3];
            },
            [&](int tm) { return row_base + tm * 16 + i16; }, f32_all, inf,
            stored ? L.f32col : nullptr);
    }
}

template <int NT, int W, int TM>
using TileLds = std::conditional_t<NT == 1, F32Lds<tile_group(1, W, TM)>,
                                   SplitLds<NT, tile_group(NT, W, TM)>>;

// One call: one workgroup per (strip of any block, 16 TM W-row tile, sketch-column
// block).
template <int NT, int W, int TM, bool GEN, bool FULL>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(NT == 1 ? 4 : 2)))
void k_gemm_mfma(const MArgs args) {
    __shared__ __attribute__((aligned(16))) TileLds<NT, W, TM> lds;
    TileId id;
    if (!mfma_tile_id<(NT > 1)>(args, id)) return;
    const int strip = id.strip;
    int b = 0;
    int64_t sib = strip;
    for (; b < args.P; ++b) {
        const int64_t sb = (args.blk[b].n + kMfmaStrip - 1) / kMfmaStrip;
        if (sib < sb) break;
        sib -= sb;
    }
    const BlockDesc& blk = args.blk[b];
    MTile t;
    t.A = static_cast<const unsigned char*>(blk.A);
    t.lda = blk.lda;
    t.n = blk.n;
    t.row0 = blk.row0;
    t.scales = blk.scales;
    t.m = args.m;
    t.k = args.k;
    t.col_begin = sib * kMfmaStrip;
    t.block_row = id.rtile * (16 * TM * W);
    t.n_base = id.nb * 16 * NT;
    t.key0 = args.key0;
    t.key1 = args.key1;
    t.col0 = args.col0;
    t.dist = args.dist;
    t.omega = args.omega;
    t.ldo = args.ldo;
    t.Y = args.Y;
    t.ldy = args.ldy;
    t.y_f64 = args.y_f64;
    t.beta = args.beta;
    t.partials = args.partials;
    t.strip = strip;
    t.single = (args.S_total == 1);
    t.opack = nullptr;
    t.opack_lo = nullptr;
    t.kpad = args.kpad;
    t.fpack = args.fpack;
    if constexpr (NT == 1) mfma_tile_f32<W, TM, GEN, FULL>(t, lds);
    else mfma_tile<NT, W, TM, GEN, FULL, mfma_packed(NT)>(t, lds);
}

// A batch of independent requests (serving): 512-row tiles of all requests, walked by a
// fixed grid in an XCD-grouped order, Omega generated in the tile.  A row's sums depend on
// neither, so each result is that of a call for the request alone.
template <int NT, bool FULL>
__global__ __launch_bounds__(kThreads) void k_gemm_mfma_batch(const BatchArgs args) {
    __shared__ __attribute__((aligned(16))) TileLds<NT, kWaves, kTM> lds;
    const int64_t T8 = (args.total_tiles + 7) / 8;
    bool first = true;
    for (int64_t v = blockIdx.x; v < 8 * T8; v += gridDim.x) {   // gridDim.x is a multiple of 8
        const int64_t tt = (v % 8) * T8 + v / 8;
        if (tt >= args.total_tiles) continue;
        int q = 0;
        while (q + 1 < args.count && tt >= args.req[q + 1].tile_begin) ++q;
        const BatchReq& rq = args.req[q];
        const int64_t lt = tt - rq.tile_begin;
        const int64_t strip = lt % rq.strips;
        const int64_t rb = (lt / rq.strips) % rq.rowblocks;
        const int nb = (int)(lt / ((int64_t)rq.strips * rq.rowblocks));
        MTile t;
        t.A = static_cast<const unsigned char*>(rq.A);
        t.lda = rq.lda;
        t.n = rq.n;
        t.row0 = rq.row0;
        t.scales = rq.scales;
        t.m = rq.m;
        t.k = rq.k;
        t.col_begin = strip * kMfmaStrip;
        t.block_row = rb * kBM;
        t.n_base = nb * 16 * NT;
        t.key0 = (uint32_t)rq.seed;
        t.key1 = (uint32_t)(rq.seed >> 32);
        t.col0 = rq.col0;
        t.dist = rq.dist;
        t.omega = nullptr;
        t.ldo = 0;
        t.Y = rq.Y;
        t.ldy = rq.ldy;
        t.y_f64 = rq.y_f64;
        t.beta = rq.beta;
        t.partials = rq.partials;
        t.strip = strip;
        t.single = (rq.strips == 1);
        t.opack = nullptr;
        t.opack_lo = nullptr;
        t.kpad = 0;
        t.fpack = nullptr;
        if (!first) lds_barrier_m();   // every wave is done with the previous tile's LDS
        first = false;
        if constexpr (NT == 1) mfma_tile_f32<kWaves, kTM, true, FULL>(t, lds);
        else mfma_tile<NT, kWaves, kTM, true, FULL>(t, lds);
    }
}

// ---------------------------------------------------------------------------
// Column-major A (element (i, j) at A + j*lda + i, the paper's storage order) on
// the same matrix cores, for k > 16: the same transposed product
// Y^T = Omega^T A^T, the Omega chunk in LDS with the same layout and reads.
// Lane (g, j) loads 16 bytes, rows 4j .. 4j + 3 of one column (a wave reads 256
// contiguous bytes of each of four columns per load), for the eight columns
// kc + 8 g .. kc + 8 g + 7 of a chunk; component q of the eight loads is the operand of
// row set {4j + q}, so a wave holds four 16 x 16 accumulator tiles of Y^T per
// N-tile, covering 64 rows.  A row's 32 entries of a chunk enter the MFMA at the
// positions they have in the row-major kernel and carry the same scale: both
// kernels form the same sums, and every A element is read once for all k
// sketch columns.
struct CmMArgs {
    const float* A;
    int64_t m, n, lda, row0;
    uint32_t key0, key1, col0;
    int dist;
    int64_t k;
    void* Y;
    int64_t ldy;
    int y_trans, y_f64, beta;
    float* partials;
    int S;                 // strips of kMfmaStrip columns
    int num_rb;            // 512-row tiles
    int64_t tiles, tiles8;
    const float* fpack;    // four or more N-tiles: the call's packed Omega (k_f32_pack)
    int64_t kpad;
};

// KC = the row-major kernel's chunk, so that the sums are the same.
// FULL (one whole chunk of columns; these tiles have 65 rows or more): every lane of a wave
// with rows issues the same loads each chunk from a valid address (a lane without rows
// reads row 0, its sums are never stored; a load past the strip's whole chunks re-reads
// one), so the compiler waits for the chunk in use alone (see mfma_tile).  ROWS4: m is
// a multiple of 4, so no lane's four rows are cut.
constexpr bool cm_full(int64_t n) { return n >= kSplitKC; }
// four floats at any float's alignment
typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));
// Packed Omega on the column-major tiles: four or more N-tiles, except eight
// without whole chunks (that kernel's registers have no room for the copy).
constexpr bool cm_packed(int nt, bool full) { return mfma_packed(nt) && (full || nt < 8); }

__device__ __forceinline__ TileOut cm_out(const CmMArgs& a, int strip) {
    TileOut o;
    o.scales = nullptr;
    o.partials = a.S == 1 ? nullptr : a.partials + (int64_t)strip * a.m * a.k;
    o.Y = a.Y;
    o.k = a.k;
    o.ldy = a.ldy;
    o.y_trans = a.y_trans;
    o.y_f64 = a.y_f64;
    o.beta = a.beta;
    return o;
}

template <int NT, int kKC, bool FULL, bool ROWS4>
__global__ __launch_bounds__(kThreads) void k_gemm_cm_mfma(const CmMArgs a) {
    constexpr int BN = 16 * NT;
    constexpr int kNS = kKC / 4;     // columns (and 16-byte loads) per lane and chunk
    // chunks generated per barrier: enough quads for every thread (1 when BN*KC/4 >= 512)
    constexpr int kG = kThreads / (kNS * BN) > 1 ? kThreads / (kNS * BN) : 1;
    static_assert(kG == 1 || kG % 2 == 0, "chunk pairs per generation group");
    __shared__ __attribute__((aligned(16))) _Float16 om[2 * kG][BN][kSplitRow];

    const int64_t id = blockIdx.x;
    const int64_t tt = (id % 8) * a.tiles8 + id / 8;       // XCD-grouped tile order
    if (tt >= a.tiles) return;
    const int strip = (int)(tt % a.S);
    const int rb = (int)((tt / a.S) % a.num_rb);
    const int nb = (int)(tt / ((int64_t)a.S * a.num_rb));

    MTile t{};
    t.row0 = a.row0;
    t.col_begin = (int64_t)strip * kMfmaStrip;
    t.n_base = nb * BN;
    t.key0 = a.key0;
    t.key1 = a.key1;
    t.col0 = a.col0;
    t.dist = a.dist;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4;
    const int j = lane & 15;
    const int w = (int)min<int64_t>(kMfmaStrip, a.n - t.col_begin);
    const int nchunks = (w + kKC - 1) / kKC;
    const int nfull = w / kKC;                              // whole chunks
    const int kb = (int)min<int64_t>(BN, a.k - t.n_base);
    const int64_t r0 = (int64_t)rb * kBM + wave * 64;      // first row of the wave
    const int64_t rl = r0 + 4 * j;                          // first row of the lane
    const bool active = r0 < a.m;                           // the wave has rows
    const bool full_rows = rl + 3 < a.m;
    // rows of the lane's group when m cuts it: the last four rows are loaded instead and
    // moved down (FULL)
    const int cut = FULL && rl < a.m && !full_rows ? (int)(a.m - rl) : 0;

    // ---- A loads: step s of chunk c is column col_begin + c*KC + g*KC/4 + s --------
    const float* acol = a.A + (t.col_begin + g * kNS) * a.lda +
                        (!FULL ? rl : cut ? a.m - 4 : rl >= a.m ? 0 : rl);
    auto load_a = [&](v4f* x, int c) {
        if constexpr (FULL) {
            const int cc = c < nfull ? c : nfull - 1;
#pragma unroll
            for (int s = 0; s < kNS; ++s)
                x[s] = *reinterpret_cast<const v4f_a4*>(acol + (int64_t)(cc * kKC + s) * a.lda);
            if (c != nfull || nfull == nchunks) return;
            asm volatile("" : "+s"(c));    // as ALoads
#pragma unroll
            for (int s = 0; s < kNS; ++s) {
                v4f v = {0.f, 0.f, 0.f, 0.f};
                if (c * kKC + g * kNS + s < w)
                    v = *reinterpret_cast<const v4f_a4*>(acol + (int64_t)(c * kKC + s) * a.lda);
                x[s] = v;
            }
#pragma unroll
            for (int s = 0; s < kNS; ++s) asm volatile("" : "+v"(x[s]));
            return;
        }
        if (!active || c >= nchunks) return;
        const int kl = c * kKC + g * kNS;
#pragma unroll
        for (int s = 0; s < kNS; ++s) {
            const float* p = acol + (int64_t)(c * kKC + s) * a.lda;
            if (full_rows && kl + s < w) {
                x[s] = *reinterpret_cast<const v4f*>(p);
            } else {
                v4f v = {0.f, 0.f, 0.f, 0.f};
                if (kl + s < w)
                    for (int q = 0; q < 4; ++q)
                        if (rl + q < a.m) v[q] = p[q];
                x[s] = v;
            }
        }
    };

    // packed route (as mfma_tile): 16-byte pieces of the tile's run of a chunk
    constexpr bool PK = cm_packed(NT, FULL);
    constexpr int PPL = BN * kKC / 4;
    constexpr int OPT = (PPL + kThreads - 1) / kThreads;
    static_assert(!PK || PPL % kThreads == 0, "whole pieces per thread");
    const int tid = threadIdx.x;
    auto om_load = [&](v4f* r, int c) {
        const int cc = c < nchunks ? c : nchunks - 1;
        const float* src = a.fpack + (((int64_t)strip * (kMfmaStrip / kKC) + cc) * a.kpad + t.n_base) * kKC;
#pragma unroll
        for (int i = 0; i < OPT; ++i)
            r[i] = *reinterpret_cast<const v4f*>(src + 4 * (tid + i * kThreads));
    };
    auto om_store = [&](const v4f* r, int slot) {
#pragma unroll
        for (int i = 0; i < OPT; ++i) {
            const int p = tid + i * kThreads;
            split_store4(om[slot][p / (kKC / 4)], (p % (kKC / 4)) * 4, r[i], 0x1p13f);
        }
    };

    if constexpr (!PK) omega_zero_pad<BN, kThreads>(om, 2 * kG, kb);
    v4f acc[4][NT];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[q][nt] = v4f{0.f, 0.f, 0.f, 0.f};
    float sc[4];                  // scale of row rl + q
    bool inf[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        sc[q] = kRowStart;
        inf[q] = false;
    }

    // a cut group's rows, loaded as the last four
    auto shift_cut = [&](v4f* x) {
        if constexpr (FULL && !ROWS4) {
            if (cut == 1) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = v4f{x[e][3], 0.f, 0.f, 0.f};
            } else if (cut == 2) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = v4f{x[e][2], x[e][3], 0.f, 0.f};
            } else if (cut == 3) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = v4f{x[e][1], x[e][2], x[e][3], 0.f};
            }
        }
    };
    h8 a0[4], a1[4], a0s[4];
    auto split = [&](v4f* x) {
        shift_cut(x);
        float y[4][8];
        float mx = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int e = 0; e < 8; ++e) y[q][e] = x[e][q] * sc[q];
            mx = absmax8(y[q], mx);
        }
        if (__builtin_expect(__any(mx > kRowLimit), 0)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float xq[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) xq[e] = x[e][q];
                const float f = rescale_row(xq, sc[q], inf[q]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[q][nt] *= f;
#pragma unroll
                for (int e = 0; e < 8; ++e) y[q][e] = x[e][q] * sc[q];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) split_a(y[q], a0[q], a1[q], a0s[q]);
    };
    auto compute = [&](int slot) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const _Float16* ob = &om[slot][nt * 16 + j][8 * g];
            const h8 b0 = *reinterpret_cast<const h8*>(ob);
            const h8 b1 = *reinterpret_cast<const h8*>(ob + kKC);
            const h8 b2 = *reinterpret_cast<const h8*>(ob + 2 * kKC);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[q][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a1[q], acc[q][nt], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[q][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b2, a0s[q], acc[q][nt], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[q][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b1, a0s[q], acc[q][nt], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[q][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b0, a0[q], acc[q][nt], 0, 0, 0);
        }
    };
    // chunk c: its A split, its registers refilled, its MFMAs
    auto consume = [&](v4f* x, int c, int slot) {
        split(x);
        load_a(x, c + (single_a(NT) ? 1 : 2));
        if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
        compute(slot);
    };

    const bool f32_all = w < kKC;             // see f32_sums
    if (!f32_all && !active) {
        // a wave without rows forms its share of Omega and leaves the units to the others
        // (at 65 .. 448 rows it would take as long as they do: tmatmul of 65536 x 80 81 us)
        if constexpr (PK) {
            v4f orr[OPT];
            om_load(orr, 0);
            om_store(orr, 0);
            om_load(orr, 1);
            lds_barrier_m();
            for (int c = 0; c < nchunks; ++c) {
                om_store(orr, (c + 1) & 1);
                om_load(orr, c + 2);
                lds_barrier_m();
            }
        } else {
            omega_group<BN, kThreads, kG, true>(t, om, 0, 0, nchunks, w, kb);
            lds_barrier_m();
            for (int cb = 0; cb < nchunks; cb += kG) {
                if (cb + kG < nchunks)
                    omega_group<BN, kThreads, kG, true>(t, om, ((cb / kG) & 1 ? 0 : kG), cb + kG,
                                                        nchunks, w, kb);
                lds_barrier_m();
            }
        }
    } else if (!f32_all) {
        v4f x0[kNS], x1[kNS];
        v4f orr[PK ? OPT : 1];
        if constexpr (PK) {
            static_assert(!PK || kG == 1, "one chunk per barrier on the packed route");
            om_load(orr, 0);
            load_a(x0, 0);
            om_store(orr, 0);
            om_load(orr, 1);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!single_a(NT)) load_a(x1, 1);
        } else {
            load_a(x0, 0);
            if constexpr (!single_a(NT)) load_a(x1, 1);
            omega_group<BN, kThreads, kG, true>(t, om, 0, 0, nchunks, w, kb);
        }
        lds_barrier_m();

        if constexpr (PK) {
            // the order of mfma_tile's packed loop
            auto step = [&](v4f* x, int c) {
                om_store(orr, (c + 1) & 1);
                om_load(orr, c + 2);
                __builtin_amdgcn_sched_barrier(0);
                consume(x, c, c & 1);
                lds_barrier_m();
            };
            if constexpr (single_a(NT)) {
                for (int c = 0; c < nchunks; ++c) step(x0, c);
            } else {
                for (int c = 0; c < nchunks; c += 2) {
                    step(x0, c);
                    if (c + 1 < nchunks) step(x1, c + 1);
                }
            }
        } else if constexpr (single_a(NT)) {
            for (int c = 0; c < nchunks; ++c) {
                if (c + 1 < nchunks)
                    omega_group<BN, kThreads, 1, true>(t, om, (c + 1) & 1, c + 1, nchunks, w, kb);
                consume(x0, c, c & 1);
                lds_barrier_m();
            }
        } else if constexpr (kG == 1) {
            for (int c = 0; c < nchunks; c += 2) {
                if (c + 1 < nchunks)
                    omega_group<BN, kThreads, 1, true>(t, om, 1, c + 1, nchunks, w, kb);
                consume(x0, c, 0);
                lds_barrier_m();
                if (c + 1 < nchunks) {
                    if (c + 2 < nchunks)
                        omega_group<BN, kThreads, 1, true>(t, om, 0, c + 2, nchunks, w, kb);
                    consume(x1, c + 1, 1);
                    lds_barrier_m();
                }
            }
        } else {
            // group u of kG chunks sits in slots (u & 1) kG ..; the next group is generated
            // into the other half while this one is consumed, one barrier per group
            for (int cb = 0; cb < nchunks; cb += kG) {
                const int half = (cb / kG) & 1;
                if (cb + kG < nchunks)
                    omega_group<BN, kThreads, kG, true>(t, om, (half ^ 1) * kG, cb + kG, nchunks, w, kb);
#pragma unroll
                for (int i = 0; i < kG; i += 2) {
                    if (cb + i < nchunks) consume(x0, cb + i, half * kG + i);
                    if (cb + i + 1 < nchunks) consume(x1, cb + i + 1, half * kG + i + 1);
                }
                lds_barrier_m();
            }
        }
    }
    // ---- lane l holds Y^T rows (sketch columns) 4g .. 4g + 3 of column j of each
    // accumulator tile: Y[rl + q][n_base + 16 nt + 4g + r] = acc[q][nt][r] ---------------
    const TileOut o = cm_out(a, strip);
    const bool vec = o.vec();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (f32_all || rl + q >= a.m || inf[q]) continue;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            emit_split(o, vec, rl + q, t.n_base + nt * 16 + 4 * g, t.n_base + kb, acc[q][nt], sc[q],
                       nullptr);
    }
    if (__syncthreads_or(f32_all || inf[0] || inf[1] || inf[2] || inf[3])) {
        t.strip = strip;
        t.m = a.m;
        t.kpad = a.kpad;
        t.fpack = a.fpack;
        f32_sums<NT, 4, kThreads, true, PK>(
            t, o, reinterpret_cast<float*>(&om[0][0][0]), w, kb, active,
            [&](float (&x)[4][8], int c) {
                v4f r[kNS];
                load_a(r, c);
                shift_cut(r);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[q][e] = r[e][q];
            },
            [&](int q) { return rl + q; }, f32_all, inf, nullptr);
    }
}

// Few rows (m <= 64; e.g. B^T of the Nystrom second product): the kernel above
// gives a tile's 64 rows to one wave, which runs all 4 x NT accumulator chains
// while the other seven idle.  Here a workgroup takes one strip and one N-tile of
// 16 sketch columns, and its waves split the work: waves 0..3 each run one chain
// (row set q = wave: rows 4j + q of lane j) with the steps, operands and order of
// the kernel above, so the results equal it (and the row-major kernel) bit for
// bit; waves 4..11 stage kSkG chunks at a time, A and the call's packed Omega,
// into the other half of a double-buffered LDS ring, with the loads of the group
// after next in flight while they store the next one.  A chain's step then waits
// on LDS only, not on a global load.  The launch always packs the call's Omega
// for this kernel (a.fpack is set).  Eight staging waves rather than four: the
// staging alone took most of the kernel's time.
constexpr int kSkG = 4;
constexpr int kSkChainThreads = 256;                       // waves 0..3
constexpr int kSkGenThreads = 512;                         // waves 4..11
constexpr int kSkThreads = kSkChainThreads + kSkGenThreads;

// ROWS: kWhole (m a multiple of 4), kCut (the group of four rows that m cuts is loaded as the
// last four and moved down on its way to LDS: with its four elements loaded one by one, behind
// branches, C = Omega^T B of 58688 x 42 took 55.5 us instead of 39.8, 50.7 on the FP32
// instruction) or kFew (m < 4: element by element).
enum { kWhole, kCut, kFew };
template <int kKC, int ROWS>
__global__ __launch_bounds__(kSkThreads) void k_gemm_cm_mfma_skinny(const CmMArgs a) {
    constexpr int BN = 16;
    constexpr int kNS = kKC / 4;
    constexpr int kGenThreads = kSkGenThreads;
    // a staged column of A: row 4j + q at [q][j], 2 floats of padding so that the
    // four lane groups of a chain's read (8 columns apart) fall on different banks
    constexpr int kAP = 66;
    constexpr int kAPieces = kSkG * kKC * 16 / kGenThreads;       // 16-byte pieces of A per thread
    constexpr int kOPieces = kSkG * BN * kKC / 4 / kGenThreads;   // and of Omega
    static_assert(kAPieces * kGenThreads == kSkG * kKC * 16 &&
                  kOPieces * kGenThreads == kSkG * BN * kKC / 4, "whole pieces per thread");
    __shared__ __attribute__((aligned(16))) _Float16 om[2 * kSkG][BN][kSplitRow];
    __shared__ float as[2 * kSkG][kKC][kAP];

    const int64_t tt = blockIdx.x;
    if (tt >= a.tiles) return;
    const int strip = (int)(tt % a.S);
    const int nb = (int)(tt / a.S);
    const int64_t col_begin = (int64_t)strip * kMfmaStrip;
    const int n_base = nb * BN;

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const bool gen_wave = wave >= 4;
    const int q = wave & 3;
    const int g = lane >> 4;
    const int j = lane & 15;
    const int w = (int)min<int64_t>(kMfmaStrip, a.n - col_begin);
    const int nchunks = (w + kKC - 1) / kKC;
    const int ngroups = (nchunks + kSkG - 1) / kSkG;
    const int kb = (int)min<int64_t>(BN, a.k - n_base);
    const int64_t rl = 4 * j;                               // first row of the lane

    // staging (waves 4..11).  Every load is issued unconditionally from a valid
    // address (chunks past the strip's last re-read it, rows past m read rows 0..3,
    // columns past the strip's end read its last column), so the compiler waits for
    // the older group only; columns past the strip's end are stored as zeros, rows
    // past m are never stored by the chains.
    const int tg = threadIdx.x - kSkChainThreads;
    // rows of the thread's group of four (the same in each of its pieces) if m cuts it
    const int left = (int)a.m - 4 * (tg & 15);
    const int cut = left > 0 && left < 4 ? left : 0;
    auto g_load = [&](int gi, v4f* xa, v4f* xo) {
#pragma unroll
        for (int t = 0; t < kAPieces; ++t) {
            const int p = tg + t * kGenThreads;
            const int ci = p / (kKC * 16);
            const int rem = p - ci * (kKC * 16);
            const int col = rem >> 4;
            const int r4 = rem & 15;
            const int c = min(gi * kSkG + ci, nchunks - 1);
            const int64_t colg = col_begin + min(c * kKC + col, w - 1);
            const float* src = a.A + colg * a.lda;
            if constexpr (ROWS == kWhole) {
                xa[t] = *reinterpret_cast<const v4f*>(src + (4 * r4 < a.m ? 4 * r4 : 0));
            } else if constexpr (ROWS == kCut) {
                xa[t] = *reinterpret_cast<const v4f_a4*>(src + (cut ? a.m - 4 : 4 * r4 < a.m ? 4 * r4 : 0));
            } else {
                v4f v = {0.f, 0.f, 0.f, 0.f};
                for (int e = 0; e < 4; ++e)
                    if (4 * r4 + e < a.m) v[e] = src[4 * r4 + e];
                xa[t] = v;
            }
        }
#pragma unroll
        for (int t = 0; t < kOPieces; ++t) {
            const int it = tg + t * kGenThreads;
            constexpr int PPC = BN * kKC / 4;                   // pieces per chunk
            const int ci = it / PPC;
            const int pc = it - ci * PPC;
            const int c = min(gi * kSkG + ci, nchunks - 1);
            const int n = pc / (kKC / 4);
            const int kl4 = (pc - n * (kKC / 4)) * 4;
            xo[t] = *reinterpret_cast<const v4f*>(
                a.fpack + (((int64_t)strip * (kMfmaStrip / kKC) + c) * a.kpad + n_base + n) * kKC + kl4);
        }
    };
    auto g_store = [&](int gi, const v4f* xa, const v4f* xo) {
        const int slot0 = (gi & 1) * kSkG;
#pragma unroll
        for (int t = 0; t < kAPieces; ++t) {
            const int p = tg + t * kGenThreads;
            const int ci = p / (kKC * 16);
            const int rem = p - ci * (kKC * 16);
            const int col = rem >> 4;
            const int r4 = rem & 15;
            const bool inside = (gi * kSkG + ci) * kKC + col < w;
            float* dst = &as[slot0 + ci][col][r4];
            v4f v = xa[t];
            if constexpr (ROWS == kCut) {
                if (cut == 1) v = v4f{v[3], 0.f, 0.f, 0.f};
                else if (cut == 2) v = v4f{v[2], v[3], 0.f, 0.f};
                else if (cut == 3) v = v4f{v[1], v[2], v[3], 0.f};
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[16 * e] = inside ? v[e] : 0.0f;
        }
#pragma unroll
        for (int t = 0; t < kOPieces; ++t) {
            const int it = tg + t * kGenThreads;
            constexpr int PPC = BN * kKC / 4;
            const int ci = it / PPC;
            const int pc = it - ci * PPC;
            const int n = pc / (kKC / 4);
            const int kl4 = (pc - n * (kKC / 4)) * 4;
            split_store4(om[slot0 + ci][n], kl4, xo[t], 0x1p13f);
        }
    };

    v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
    float sc = kRowStart;         // scale of row rl + q
    bool inf = false;
    auto chain_group = [&](int gi) {
        const int slot0 = (gi & 1) * kSkG;
#pragma unroll
        for (int cc = 0; cc < kSkG; ++cc) {
            if (gi * kSkG + cc < nchunks) {
                const _Float16* ob = &om[slot0 + cc][j][8 * g];
                const h8 b0 = *reinterpret_cast<const h8*>(ob);
                const h8 b1 = *reinterpret_cast<const h8*>(ob + kKC);
                const h8 b2 = *reinterpret_cast<const h8*>(ob + 2 * kKC);
                const float* ab = &as[slot0 + cc][g * kNS][16 * q + j];
                float x[kNS], y[kNS];
#pragma unroll
                for (int s = 0; s < kNS; ++s) {
                    x[s] = ab[s * kAP];
                    y[s] = x[s] * sc;
                }
                if (__builtin_expect(__any(absmax8(y, 0.0f) > kRowLimit), 0)) {
                    acc *= rescale_row(x, sc, inf);
#pragma unroll
                    for (int s = 0; s < kNS; ++s) y[s] = x[s] * sc;
                }
                h8 a0, a1, a0s;
                split_a(y, a0, a1, a0s);
                acc = split_mfma(b0, b1, b2, a0, a1, a0s, acc);
            }
        }
    };

    const bool f32_all = w < kKC;             // see f32_sums; the strip's only chunk
    v4f ra[kAPieces], ro[kOPieces], rb[kAPieces], rbo[kOPieces];
    if (gen_wave) {
        g_load(0, ra, ro);
        g_store(0, ra, ro);
        g_load(min(1, ngroups - 1), ra, ro);
    }
    lds_barrier_m();
    // group gi: the chains use slot gi & 1; the stagers store group gi + 1 (held in
    // cur) into the other slot after issuing the loads of group gi + 2 into nxt
    auto iter = [&](int gi, v4f* cur_a, v4f* cur_o, v4f* nxt_a, v4f* nxt_o) {
        if (gen_wave) {
            g_load(min(gi + 2, ngroups - 1), nxt_a, nxt_o);
            if (gi + 1 < ngroups) g_store(gi + 1, cur_a, cur_o);
        } else {
            chain_group(gi);
        }
        lds_barrier_m();
    };
    for (int gi = 0; gi < ngroups; gi += 2) {
        iter(gi, ra, ro, rb, rbo);
        if (gi + 1 < ngroups) iter(gi + 1, rb, rbo, ra, ro);
    }
    // lane (g, j) of a chain holds Y^T rows (sketch columns) 4g .. 4g + 3 of column j of
    // the tile: Y[rl + q][n_base + 4g + r] = acc[r]
    const TileOut o = cm_out(a, strip);
    const int64_t row = rl + q;
    if (!gen_wave && row < a.m && !inf && !f32_all)
        emit_split(o, o.vec(), row, n_base + 4 * g, n_base + kb, acc, sc, nullptr);
    if (__syncthreads_or(!gen_wave && (f32_all || inf))) {
        MTile t{};
        t.m = a.m;
        t.n_base = n_base;
        t.strip = strip;
        t.kpad = a.kpad;
        t.fpack = a.fpack;
        f32_sums<1, 1, kSkThreads, true, true>(
            t, o, reinterpret_cast<float*>(&om[0][0][0]), w, kb, !gen_wave,
            [&](float (&x)[1][8], int c) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int kl = c * kKC + 8 * g + e;
                    x[0][e] = kl < w && row < a.m ? a.A[(col_begin + kl) * a.lda + row] : 0.0f;
                }
            },
            [&](int) { return row; }, f32_all, {inf}, nullptr);
    }
}

template <int NT, int KC>
hipError_t launch_cm_mfma_nt(const CmMArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)(8 * a.tiles8));
    if (!cm_full(a.n))
        hipLaunchKernelGGL((k_gemm_cm_mfma<NT, KC, false, false>), grid, dim3(kThreads), 0, s, a);
    else if (a.m % 4 == 0)
        hipLaunchKernelGGL((k_gemm_cm_mfma<NT, KC, true, true>), grid, dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL((k_gemm_cm_mfma<NT, KC, true, false>), grid, dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Low-precision A (BF16, or FP8-E4M3 widened to BF16 exactly) on the BF16
// matrix cores: v_mfma_f32_16x16x32_bf16, FP32 accumulate.  Omega is split into
// two BF16 terms, hi = bf16(w) and lo = bf16(w - hi), and each step runs two
// MFMAs (A*hi, then A*lo): |w - hi - lo| <= 2^-16 |w|, far below the storage
// error of A, so the product carries A's quantisation only.  The workgroup
// is W waves x 64 rows sharing each generated Omega chunk (a run of
// contraction columns): the more rows, the less generation per A element, which matters
// because a byte of FP8 holds four times the elements of a byte of FP32.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// Contraction columns per chunk: 128 bytes of every row (BF16: 64 columns,
// FP8: 128), 32 bytes per lane, so a row is read in whole 128-byte lines
// (measured: 64-byte runs cost FP8 a quarter of its rate; 256-byte runs gain
// nothing and cost registers).
constexpr int lp_kc(int adt) { return adt == 2 ? 128 : 64; }
constexpr int lp_row(int adt) { return lp_kc(adt) + 8; }   // bf16 per LDS column (+8 pad)
static_assert(64 * kLpBatchWaves == kLpBatchRows, "batch tile rows");

__device__ __forceinline__ uint32_t bf16_rne_bits(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// Omega value -> (hi, lo) BF16 bit patterns; z - hi is exact in FP32.
__device__ __forceinline__ void split_bf16(float z, uint16_t& hi, uint16_t& lo) {
    const uint32_t h = bf16_rne_bits(z);
    hi = (uint16_t)h;
    lo = (uint16_t)bf16_rne_bits(z - __uint_as_float(h << 16));
}

// 4 FP8-E4M3 codes (one word) -> 4 BF16 in two words, element order kept (exact:
// 4 significant bits).  PACKED: one gfx950 packed conversion per pair (scale 1);
// otherwise through FP32 and a repack.  Both give the same bits; measured on
// 32768^2, the packed form is 3% faster with four N-tiles and 3% slower with
// one (whose kernel sits at the 128-register cap).
template <bool PACKED>
__device__ __forceinline__ void fp8x4_to_bf16(uint32_t w, uint32_t& lo2, uint32_t& hi2) {
    if constexpr (PACKED) {
        lo2 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w, 1.0f, false));
        hi2 = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w, 1.0f, true));
    } else {
        const auto a = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false);
        const auto b = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
        lo2 = (__float_as_uint(a[1]) & 0xFFFF0000u) | (__float_as_uint(a[0]) >> 16);
        hi2 = (__float_as_uint(b[1]) & 0xFFFF0000u) | (__float_as_uint(b[0]) >> 16);
    }
}

// ---- Omega of a whole call, split and laid out for the low-precision tiles ----
// Every row tile of a strip multiplies the same Omega chunks, so a call's
// Omega (hi, lo) is formed once, before the product, instead of once per
// 64W-row tile (a 32768-row FP8 call has 64 tiles per strip).  Layout, one
// plane for hi and one for lo: chunk gc = strip * (kLpStrip / KC) + c, then
// sketch column n in [0, kpad), then contraction column kl in [0, KC):
// element ((gc * kpad + n) * KC + kl).  A tile's BN columns of a chunk are
// then one contiguous run of BN * KC values.  Entries past the strip's last
// column and sketch columns >= k hold zero; the values are those the fused
// generation writes into LDS, so both routes give the same sums bit for bit.

// sketch columns per packing workgroup: 16 gives each compute unit several
// workgroups to interleave (the work is a chain of dependent arithmetic)
constexpr int kPackRows = 16;

// grid (chunks of all strips, ceil(kpad / 16)); 256 threads
template <int ADT, bool GEN>
__global__ __launch_bounds__(256) void k_lp_pack(const PackArgs a) {
    constexpr int KC = lp_kc(ADT);
    constexpr int R = lp_row(ADT);
    constexpr int CPS = kLpStrip / KC;
    __shared__ __attribute__((aligned(16))) uint16_t sh[2][kPackRows][R];
    const int tid = threadIdx.x;
    const int64_t gc = blockIdx.x;
    const int64_t strip = gc / CPS;
    const int c = (int)(gc - strip * CPS);
    int b = 0;
    int64_t sib = strip;
    for (; b < a.P; ++b) {
        const int64_t sb = (a.blk[b].n + kLpStrip - 1) / kLpStrip;
        if (sib < sb) break;
        sib -= sb;
    }
    const int64_t col_begin = sib * kLpStrip;
    const int w = (int)min<int64_t>(kLpStrip, a.blk[b].n - col_begin);
    if (c * KC >= w) return;                      // past the strip's end: never read
    const int kvalid = min(KC, w - c * KC);
    const int nb0 = blockIdx.y * kPackRows;
    const int kb = (int)min<int64_t>(kPackRows, a.k - nb0);   // <= 0: all zero
    static_assert((2 * kPackRows * R) % 8 == 0, "whole 16-byte pieces");
    for (int it = tid; it < 2 * kPackRows * R / 8; it += 256)
        reinterpret_cast<v4u*>(&sh[0][0][0])[it] = v4u{0u, 0u, 0u, 0u};
    __syncthreads();
    if constexpr (GEN) {
        const int64_t g0 = a.blk[b].row0 + col_begin + (int64_t)c * KC;
        const int64_t q_lo = g0 >> 2;
        const int nq = (int)(((g0 + KC - 1) >> 2) - q_lo + 1);
        const int items = kb > 0 ? nq * kb : 0;
        for (int it = tid; it < items; it += 256) {
            const int qi = it / kb;
            const int n = it - qi * kb;
            const float4 z = omega4_dist((uint64_t)(q_lo + qi), a.col0 + (uint32_t)(nb0 + n),
                                         a.key0, a.key1, a.dist);
            const int kl0 = (int)(4 * (q_lo + qi) - g0);
            const float zz[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int kl = kl0 + u;
                if (kl >= 0 && kl < kvalid) split_bf16(zz[u], sh[0][n][kl], sh[1][n][kl]);
            }
        }
    } else {
        const int items = kb > 0 ? kvalid * kb : 0;
        for (int it = tid; it < items; it += 256) {
            const int kl = it / kb;
            const int n = it - kl * kb;
            split_bf16(a.omega[(col_begin + (int64_t)c * KC + kl) * a.ldo + nb0 + n],
                       sh[0][n][kl], sh[1][n][kl]);
        }
    }
    __syncthreads();
    const int rows = (int)min<int64_t>(kPackRows, a.kpad - nb0);
    const int pieces = rows * (KC / 8);           // 16-byte pieces per plane
    for (int it = tid; it < 2 * pieces; it += 256) {
        const int pl = it >= pieces;
        const int q = it - pl * pieces;
        const int n = q / (KC / 8);
        const int kl8 = (q - n * (KC / 8)) * 8;
        uint16_t* dst = static_cast<uint16_t*>(pl ? a.lo : a.hi) + ((gc * a.kpad + nb0 + n) * KC + kl8);
        *reinterpret_cast<v4u*>(dst) = *reinterpret_cast<const v4u*>(&sh[pl][n][kl8]);
    }
}

// FULL: whole chunks only, unconditional A loads (as in mfma_tile).
// PK: Omega chunks copied from the call's packed Omega (k_lp_pack) instead of
// generated or split here; the copy of chunk c + 2 is issued ahead of the A
// loads of chunk c + 2, so waiting for it leaves those in flight.
template <int NT, int ADT, int W, int TM, bool GEN, bool FULL = false, bool PK = false>
__device__ __forceinline__ void lp_tile(const MTile& t, uint16_t (*oh)[16 * NT][lp_row(ADT)],
                                        uint16_t (*ol)[16 * NT][lp_row(ADT)]) {
    constexpr int BN = 16 * NT;
    constexpr int TH = 64 * W;
    constexpr int KC = lp_kc(ADT);
    constexpr int KG = KC / 4;            // columns of a lane group per chunk
    constexpr int V = KC / 32;            // MFMA steps per chunk
    constexpr int es = ADT == 1 ? 2 : 1;
    constexpr int RW = 2;                 // 16-byte raw A words per lane and M-tile
    static_assert(KG * es == 16 * RW && kLpStrip % KC == 0, "chunk geometry");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int g = lane >> 4;
    const int i16 = lane & 15;

    const int w = (int)min<int64_t>(kLpStrip, t.n - t.col_begin);
    const int nchunks = (w + KC - 1) / KC;
    const int64_t row_base = t.block_row + wave * (TM * 16);
    const int kb = (int)min<int64_t>(BN, t.k - t.n_base);

    // ---- A: lane (g, i) holds columns kc + KG g .. kc + KG g + KG - 1 of row i ------
    const int64_t ldab = t.lda * es;
    const unsigned char* arow[TM];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int64_t r = min<int64_t>(row_base + tm * 16 + i16, t.m - 1);
        arow[tm] = t.A + r * ldab + (t.col_begin + KG * g) * es;
    }
    // raw A of a chunk, RW words per lane and M-tile; FP8 is widened to BF16
    // only when the chunk is consumed, so the loads stay in flight behind the
    // current chunk's MFMAs
    auto load_a = [&](v4u (*a)[RW], int c) {
        if constexpr (FULL) {
            const int cc = c < nchunks ? c : nchunks - 1;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const unsigned char* p = arow[tm] + (int64_t)cc * KC * es;
#pragma unroll
                for (int v = 0; v < RW; ++v) a[tm][v] = *reinterpret_cast<const v4u*>(p + 16 * v);
            }
            return;
        }
        if (c >= nchunks) return;
        const int kl = c * KC + KG * g;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const unsigned char* p = arow[tm] + (int64_t)c * KC * es;
            if (kl + KG - 1 < w) {
#pragma unroll
                for (int v = 0; v < RW; ++v) a[tm][v] = *reinterpret_cast<const v4u*>(p + 16 * v);
            } else {
                uint32_t wd[4 * RW];
#pragma unroll
                for (int q = 0; q < 4 * RW; ++q) wd[q] = 0u;
                for (int e = 0; e < KG; ++e) {
                    if (kl + e < w) {
                        const uint32_t v = ADT == 1 ? (uint32_t)reinterpret_cast<const uint16_t*>(p)[e]
                                                    : (uint32_t)p[e];
                        const int byte = e * es;
                        wd[byte >> 2] |= v << (8 * (byte & 3));
                    }
                }
#pragma unroll
                for (int v = 0; v < RW; ++v)
                    a[tm][v] = v4u{wd[4 * v], wd[4 * v + 1], wd[4 * v + 2], wd[4 * v + 3]};
            }
        }
    };
    // the 8-element BF16 operand of MFMA step v (columns KG g + 8v .. + 7 of the lane)
    auto operand = [&](const v4u* raw, int v) -> v4u {
        if constexpr (ADT == 1) {
            return raw[v];
        } else {
            const v4u r = raw[v >> 1];     // 16 FP8 = two steps per word
            const int q = 2 * (v & 1);
            uint32_t o[4];
            fp8x4_to_bf16<(NT > 1)>(r[q], o[0], o[1]);
            fp8x4_to_bf16<(NT > 1)>(r[q + 1], o[2], o[3]);
            return v4u{o[0], o[1], o[2], o[3]};
        }
    };

    // ---- Omega chunk -> LDS as (hi, lo) ------------------------------------------
    if constexpr (!PK) {
        for (int it = tid; it < 2 * BN * lp_row(ADT); it += TH) {
            const int n = (it / lp_row(ADT)) % BN;
            if (n >= kb) {
                (&oh[0][0][0])[it] = 0;
                (&ol[0][0][0])[it] = 0;
            }
        }
    }
    // packed route: 16-byte pieces of the tile's run of a chunk (both planes),
    // OPT per thread; chunk indices past the last are clamped (a re-read of
    // valid memory whose copy lands in the LDS buffer no step reads next)
    constexpr int PPL = BN * KC / 8;              // pieces per plane
    constexpr int OPT = (2 * PPL + TH - 1) / TH;
    auto om_load = [&](v4u* r, int c) {
        const int cc = c < nchunks ? c : nchunks - 1;
        const int64_t off = ((t.strip * (kLpStrip / KC) + cc) * t.kpad + t.n_base) * KC;
#pragma unroll
        for (int j = 0; j < OPT; ++j) {
            const int p = min(tid + j * TH, 2 * PPL - 1);
            const int pl = p >= PPL;
            const uint16_t* src = (pl ? t.opack_lo : t.opack) + off + (p - pl * PPL) * 8;
            r[j] = *reinterpret_cast<const v4u*>(src);
        }
    };
    auto om_store = [&](const v4u* r, int c) {
        const int buf = c & 1;
#pragma unroll
        for (int j = 0; j < OPT; ++j) {
            const int p = min(tid + j * TH, 2 * PPL - 1);
            const int pl = p >= PPL;
            const int q = p - pl * PPL;
            const int n = q / (KC / 8);
            const int kl8 = (q - n * (KC / 8)) * 8;
            *reinterpret_cast<v4u*>(pl ? &ol[buf][n][kl8] : &oh[buf][n][kl8]) = r[j];
        }
    };
    auto make_chunk = [&](int c) {
        const int buf = c & 1;
        const int kvalid = min(KC, w - c * KC);
        if constexpr (GEN) {
            const int64_t g0 = t.row0 + t.col_begin + (int64_t)c * KC;
            const int64_t q_lo = g0 >> 2;
            const int nq = (int)(((g0 + KC - 1) >> 2) - q_lo + 1);
            const int items = nq * kb;
            for (int it = tid; it < items; it += TH) {
                const int qi = it / kb;
                const int n = it - qi * kb;
                const float4 z = omega4_dist((uint64_t)(q_lo + qi), t.col0 + (uint32_t)(t.n_base + n),
                                             t.key0, t.key1, t.dist);
                const int kl0 = (int)(4 * (q_lo + qi) - g0);
                const float zz[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int kl = kl0 + u;
                    if (kl >= 0 && kl < KC) {
                        uint16_t h = 0, l = 0;
                        if (kl < kvalid) split_bf16(zz[u], h, l);
                        oh[buf][n][kl] = h;
                        ol[buf][n][kl] = l;
                    }
                }
            }
        } else {
            for (int it = tid; it < KC * kb; it += TH) {
                const int kl = it / kb;
                const int n = it - kl * kb;
                uint16_t h = 0, l = 0;
                if (kl < kvalid)
                    split_bf16(t.omega[(t.col_begin + (int64_t)c * KC + kl) * t.ldo + t.n_base + n],
                               h, l);
                oh[buf][n][kl] = h;
                ol[buf][n][kl] = l;
            }
        }
    };

    v4f acc[TM][NT];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[tm][nt] = v4f{0.f, 0.f, 0.f, 0.f};

    v4u a0[TM][RW], a1[TM][RW];
    v4u orr[PK ? OPT : 1];
    if constexpr (PK) {
        load_a(a0, 0);
        om_load(orr, 0);
        om_store(orr, 0);
        om_load(orr, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_a(a1, 1);
    } else {
        load_a(a0, 0);
        load_a(a1, 1);
        make_chunk(0);
    }
    lds_barrier_m();

    auto compute = [&](v4u (*a)[RW], int c) {
        const int buf = c & 1;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            v4u op[TM];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) op[tm] = operand(a[tm], v);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const v4u bh = *reinterpret_cast<const v4u*>(&oh[buf][nt * 16 + i16][KG * g + 8 * v]);
                const v4u bl = *reinterpret_cast<const v4u*>(&ol[buf][nt * 16 + i16][KG * g + 8 * v]);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    const v8bf av = __builtin_bit_cast(v8bf, op[tm]);
                    acc[tm][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        av, __builtin_bit_cast(v8bf, bh), acc[tm][nt], 0, 0, 0);
                    acc[tm][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        av, __builtin_bit_cast(v8bf, bl), acc[tm][nt], 0, 0, 0);
                }
            }
        }
    };

    if constexpr (PK) {
        // step c: chunk c + 1's Omega to LDS, chunk c + 2's Omega issued, chunk c's
        // MFMAs, chunk c + 2's A issued (the same summation order as below)
        for (int c = 0; c < nchunks; c += 2) {
            om_store(orr, c + 1);
            om_load(orr, c + 2);
            __builtin_amdgcn_sched_barrier(0);
            compute(a0, c);
            load_a(a0, c + 2);
            if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
            lds_barrier_m();
            om_store(orr, c + 2);
            om_load(orr, c + 3);
            __builtin_amdgcn_sched_barrier(0);
            if (c + 1 < nchunks) compute(a1, c + 1);
            load_a(a1, c + 3);
            if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);
            lds_barrier_m();
        }
    } else if constexpr (FULL) {
        // the same order with every load issued (and kept ahead of the next chunk's work)
        for (int c = 0; c < nchunks; c += 2) {
            if (c + 1 < nchunks) make_chunk(c + 1);
            compute(a0, c);
            load_a(a0, c + 2);
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier_m();
            if (c + 2 < nchunks) make_chunk(c + 2);
            if (c + 1 < nchunks) compute(a1, c + 1);
            load_a(a1, c + 3);
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier_m();
        }
    } else {
        for (int c = 0; c < nchunks; c += 2) {
            if (c + 1 < nchunks) make_chunk(c + 1);
            compute(a0, c);
            load_a(a0, c + 2);
            lds_barrier_m();
            if (c + 1 < nchunks) {
                if (c + 2 < nchunks) make_chunk(c + 2);
                compute(a1, c + 1);
                load_a(a1, c + 3);
                lds_barrier_m();
            }
        }
    }
    store_tile<NT, TM>(t, acc, row_base, kb, g, i16);
}

// One call: one workgroup per (strip of any block, 16 TM W-row tile, sketch-column
// block), in the XCD-grouped order of mfma_tile_id.
// One-N-tile, 4-wave workgroups are kept within 128 registers so that four of
// them share a compute unit (a 32768-row FP8 launch is exactly four per unit;
// with three, a quarter of the tiles run as a tail on an underfilled chip).
constexpr int lp_min_waves(int nt, int w, int tm) { return nt == 1 && w == 4 && tm == kTM ? 4 : 1; }

// Omega from the call's packed copy with more than one N-tile; one N-tile
// generates (or splits) its chunks in the tile, as the 128 registers of its
// 4-wave workgroups hold no staging registers besides.
constexpr bool lp_packed(int nt) { return nt > 1; }

template <int NT, int ADT, int W, int TM, bool GEN, bool FULL>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(lp_min_waves(NT, W, TM))))
void k_gemm_mfma_lp(const MArgs args) {
    __shared__ __attribute__((aligned(16))) uint16_t oh[2][16 * NT][lp_row(ADT)];
    __shared__ __attribute__((aligned(16))) uint16_t ol[2][16 * NT][lp_row(ADT)];
    TileId id;
    if (!mfma_tile_id<true>(args, id)) return;
    const int strip = id.strip;
    int b = 0;
    int64_t sib = strip;
    for (; b < args.P; ++b) {
        const int64_t sb = (args.blk[b].n + kLpStrip - 1) / kLpStrip;
        if (sib < sb) break;
        sib -= sb;
    }
    const BlockDesc& blk = args.blk[b];
    MTile t;
    t.A = static_cast<const unsigned char*>(blk.A);
    t.lda = blk.lda;
    t.n = blk.n;
    t.row0 = blk.row0;
    t.scales = blk.scales;
    t.m = args.m;
    t.k = args.k;
    t.col_begin = sib * kLpStrip;
    t.block_row = id.rtile * (16 * TM * W);
    t.n_base = id.nb * 16 * NT;
    t.key0 = args.key0;
    t.key1 = args.key1;
    t.col0 = args.col0;
    t.dist = args.dist;
    t.omega = args.omega;
    t.ldo = args.ldo;
    t.Y = args.Y;
    t.ldy = args.ldy;
    t.y_f64 = args.y_f64;
    t.beta = args.beta;
    t.partials = args.partials;
    t.strip = strip;
    t.single = (args.S_total == 1);
    t.opack = args.opack;
    t.opack_lo = args.opack_lo;
    t.kpad = args.kpad;
    t.fpack = nullptr;
    lp_tile<NT, ADT, W, TM, GEN, FULL, lp_packed(NT)>(t, oh, ol);
}

// Batch of requests of one class (serving); rows per tile = kLpBatchRows.
template <int NT, int ADT>
__global__ __launch_bounds__(64 * kLpBatchWaves) void k_gemm_mfma_lp_batch(const BatchArgs args) {
    __shared__ __attribute__((aligned(16))) uint16_t oh[2][16 * NT][lp_row(ADT)];
    __shared__ __attribute__((aligned(16))) uint16_t ol[2][16 * NT][lp_row(ADT)];
    const int64_t T8 = (args.total_tiles + 7) / 8;
    bool first = true;
    for (int64_t v = blockIdx.x; v < 8 * T8; v += gridDim.x) {   // gridDim.x is a multiple of 8
        const int64_t tt = (v % 8) * T8 + v / 8;
        if (tt >= args.total_tiles) continue;
        int q = 0;
        while (q + 1 < args.count && tt >= args.req[q + 1].tile_begin) ++q;
        const BatchReq& rq = args.req[q];
        const int64_t lt = tt - rq.tile_begin;
        const int64_t strip = lt % rq.strips;
        const int64_t rb = (lt / rq.strips) % rq.rowblocks;
        const int nb = (int)(lt / ((int64_t)rq.strips * rq.rowblocks));
        MTile t;
        t.A = static_cast<const unsigned char*>(rq.A);
        t.lda = rq.lda;
        t.n = rq.n;
        t.row0 = rq.row0;
        t.scales = rq.scales;
        t.m = rq.m;
        t.k = rq.k;
        t.col_begin = strip * kLpStrip;
        t.block_row = rb * kLpBatchRows;
        t.n_base = nb * 16 * NT;
        t.key0 = (uint32_t)rq.seed;
        t.key1 = (uint32_t)(rq.seed >> 32);
        t.col0 = rq.col0;
        t.dist = rq.dist;
        t.omega = nullptr;
        t.ldo = 0;
        t.Y = rq.Y;
        t.ldy = rq.ldy;
        t.y_f64 = rq.y_f64;
        t.beta = rq.beta;
        t.partials = rq.partials;
        t.strip = strip;
        t.single = (rq.strips == 1);
        t.opack = nullptr;
        t.opack_lo = nullptr;
        t.kpad = 0;
        t.fpack = nullptr;
        if (!first) lds_barrier_m();
        first = false;
        lp_tile<NT, ADT, kLpBatchWaves, kTM, true>(t, oh, ol);
    }
}

template <int NT, int ADT, int W, int TM, bool GEN>
hipError_t launch_lp(const MArgs& args, hipStream_t s) {
    MArgs a = args;
    a.nrt = (a.m + 16 * TM * W - 1) / (16 * TM * W);
    const dim3 grid = mfma_grid(a);
    // whole chunks: unconditional loads (one N-tile measured 5-8% slower with them: its
    // 4-wave, 128-register tiles already keep enough loads in flight)
    bool full = NT > 1;
    for (int b = 0; b < a.P; ++b) full = full && a.blk[b].n % lp_kc(ADT) == 0;
    if (full)
        hipLaunchKernelGGL((k_gemm_mfma_lp<NT, ADT, W, TM, GEN, true>), grid, dim3(64 * W), 0, s, a);
    else
        hipLaunchKernelGGL((k_gemm_mfma_lp<NT, ADT, W, TM, GEN, false>), grid, dim3(64 * W), 0, s, a);
    return hipGetLastError();
}

template <int NT, int ADT, bool GEN>
hipError_t dispatch_lp_w(int rows, const MArgs& a, hipStream_t s) {
    switch (rows) {
    case 64: return launch_lp<NT, ADT, 4, 1, GEN>(a, s);
    case 128: return launch_lp<NT, ADT, 8, 1, GEN>(a, s);
    case 256: return launch_lp<NT, ADT, 4, 4, GEN>(a, s);
    default: return launch_lp<NT, ADT, 8, 4, GEN>(a, s);
    }
}

// packed tiles do not look at GEN (the packing kernel did): one instantiation
template <int ADT>
hipError_t dispatch_lp(int nt, bool gen, int rows, const MArgs& a, hipStream_t s) {
    static_assert(!lp_packed(1) && lp_packed(2) && lp_packed(4), "routes below");
    switch (nt) {
    case 1: return gen ? dispatch_lp_w<1, ADT, true>(rows, a, s)
                       : dispatch_lp_w<1, ADT, false>(rows, a, s);
    case 2: return dispatch_lp_w<2, ADT, true>(rows, a, s);
    default: return dispatch_lp_w<4, ADT, true>(rows, a, s);
    }
}

template <int NT, int W, int TM, bool GEN, bool FULL>
hipError_t launch_m_tile(const MArgs& args, hipStream_t s) {
    // packed tiles do not look at GEN (the packing kernel did): one instantiation
    constexpr bool G = mfma_packed(NT) || GEN;
    MArgs a = args;
    a.nrt = (a.m + 16 * TM * W - 1) / (16 * TM * W);
    hipLaunchKernelGGL((k_gemm_mfma<NT, W, TM, G, FULL>), mfma_grid(a), dim3(64 * W), 0, s, a);
    return hipGetLastError();
}

template <int NT, bool GEN>
hipError_t launch_m(int rows, const MArgs& a, hipStream_t s) {
    bool full = true, whole = true, lines = true;
    for (int b = 0; b < a.P; ++b) {
        lines = lines && a.blk[b].lda % 32 == 0 && ((uintptr_t)a.blk[b].A & 127) == 0;
        full = full && (a.blk[b].n >= kSplitKC || a.blk[b].n == 0);
        whole = whole && a.blk[b].n % kSplitKC == 0;
    }
    if (full && rows == 64) return launch_m_tile<NT, 4, 1, GEN, true>(a, s);
    if (full && rows == 128) return launch_m_tile<NT, 8, 1, GEN, true>(a, s);
    // 25 to 32 columns on rows that are not whole 128-byte lines: two 256-row tiles a compute
    // unit (120 registers) overlap one's generation with the other's twice as many line
    // requests, one 512-row tile does not (k = 28: 40000 x 7001 448 us against 325, 60000 x
    // 16388 925 against 881, 20000 x 9988 237 against 220; on whole lines 60000 x 16384 736
    // against 758)
    const bool half = NT == 2 && a.k > 24 && !lines;
    if (full && (rows == 256 || (rows == kBM && half))) return launch_m_tile<NT, 8, 2, GEN, true>(a, s);
    // one N-tile: whole chunks only (with a ragged end the unconditional loads measured
    // 166 us against 158 for the per-lane path, 20011 x 9973 at k = 16)
    return (NT == 1 ? whole : full) ? launch_m_tile<NT, 8, 4, GEN, true>(a, s)
                                    : launch_m_tile<NT, 8, 4, GEN, false>(a, s);
}

template <bool GEN>
hipError_t dispatch_m(int nt, int rows, const MArgs& a, hipStream_t s) {
    switch (nt) {
    case 1: return launch_m<1, GEN>(rows, a, s);
    case 2: return launch_m<2, GEN>(rows, a, s);
    case 4: return launch_m<4, GEN>(rows, a, s);
    default: return launch_m<8, GEN>(rows, a, s);
    }
}

}  // namespace

// N-tiles (of 16 sketch columns) per workgroup for a sketch of width k.
int mfma_ntiles(int64_t k) { return k <= 16 ? 1 : k <= 32 ? 2 : k <= 64 ? 4 : 8; }

namespace {

// workspace of a packed route: [strip partials (more than one strip)]
// [256-B aligned: the packed Omega planes]
size_t pack_offset(int64_t m, int64_t strips, int64_t k) {
    return (gemm_workspace_bytes(m, strips, k) + 255) / 256 * 256;
}

int64_t mfma_kpad(int64_t k) {
    const int64_t BN = 16 * mfma_ntiles(k);
    return (k + BN - 1) / BN * BN;
}

size_t f32_plane_elems(int64_t strips, int64_t k) {
    return (size_t)strips * (size_t)kMfmaStrip * (size_t)mfma_kpad(k);
}

}  // namespace

// Rows per tile of the FP32 kernel: 512 (8 waves of 64 rows, which share each Omega chunk),
// halved down to 64 while those tiles would fill half the compute units at most.  A strip's
// 64 chunks follow one another, so a call with few tiles takes as long as one tile, and a
// smaller tile does less per chunk.  With 512- or 256-row tiles of 64 rows a wave (before)
// and with this rule: 5000 x 5000 at k = 64 124 and 59 us, 2000 x 3000 at k = 16 86 and 43,
// at k = 24 about 95 and 80, 10000 x 2000 at k = 130 558 (FP32 instruction) and 86.
static int mfma_rows(int64_t m, int64_t strips, int64_t nblk) {
    int rows = kBM;
    while (rows > 64 && 2 * strips * ((m + rows - 1) / rows) * nblk <= device_cus()) rows /= 2;
    return rows;
}

hipError_t launch_gemm_mfma(const GemmLaunch& g) {
    const int nt = mfma_ntiles(g.k);
    const int64_t BN = 16 * nt;
    const int64_t nblk = (g.k + BN - 1) / BN;
    int64_t S = 0;
    for (int b = 0; b < g.P; ++b) S += (g.blk[b].n + kMfmaStrip - 1) / kMfmaStrip;
    PackArgs pk{};
    if (mfma_packed(nt)) {
        pk.hi = static_cast<unsigned char*>(g.workspace) + pack_offset(g.m, S, g.k);
        pk.k = g.k;
        pk.kpad = mfma_kpad(g.k);
        pk.key0 = (uint32_t)g.seed;
        pk.key1 = (uint32_t)(g.seed >> 32);
        pk.col0 = g.col0;
        pk.dist = g.dist;
        pk.omega = g.omega;
        pk.ldo = g.ldo;
        pk.P = g.P;
        for (int b = 0; b < g.P; ++b) pk.blk[b] = g.blk[b];
    }
    MArgs a{};
    a.fpack = static_cast<const float*>(pk.hi);
    a.kpad = pk.kpad;
    a.m = g.m;
    a.k = g.k;
    a.ldy = g.ldy;
    a.ldo = g.ldo;
    a.omega = g.omega;
    a.Y = g.Y;
    a.partials = S > 1 ? static_cast<float*>(g.workspace) : nullptr;
    a.key0 = (uint32_t)g.seed;
    a.key1 = (uint32_t)(g.seed >> 32);
    a.col0 = g.col0;
    a.dist = g.dist;
    a.P = g.P;
    a.S_total = (int)S;
    a.y_f64 = g.y_f64;
    a.beta = g.beta;
    for (int b = 0; b < g.P; ++b) a.blk[b] = g.blk[b];
    a.nblk = (int)nblk;
    const int rows = mfma_rows(g.m, S, nblk);
    const TraceEvents& tr = g.trace;
    if (tr.begin) (void)hipEventRecord(tr.begin, g.stream);
    if (mfma_packed(nt)) {
        const dim3 pgrid((unsigned)(S * (kMfmaStrip / kSplitKC) / kF32PackChunks),
                         (unsigned)((pk.kpad + kF32PackRows - 1) / kF32PackRows));
        if (pk.omega)
            hipLaunchKernelGGL((k_f32_pack<false>), pgrid, dim3(256), 0, g.stream, pk);
        else
            hipLaunchKernelGGL((k_f32_pack<true>), pgrid, dim3(256), 0, g.stream, pk);
        const hipError_t pe = hipGetLastError();
        if (pe != hipSuccess) return pe;
    }
    hipError_t e = (g.omega == nullptr) ? dispatch_m<true>(nt, rows, a, g.stream)
                                        : dispatch_m<false>(nt, rows, a, g.stream);
    if (e != hipSuccess) return e;
    if (tr.mid) (void)hipEventRecord(tr.mid, g.stream);
    if (S > 1) e = launch_reduce_partials(a.partials, (int)S, g.m, g.k, g.Y, g.y_f64, g.ldy,
                                          g.beta, g.stream);
    if (tr.end) (void)hipEventRecord(tr.end, g.stream);
    return e;
}

namespace {

template <int NT, bool FULL>
hipError_t run_mfma_batch_f(const BatchArgs& a, int grid, hipStream_t s) {
    static const int per_cu = [] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_gemm_mfma_batch<NT, FULL>, kThreads,
                                                         0) != hipSuccess)
            n = 1;
        return n;
    }();
    grid = batch_grid(per_cu, a.total_tiles, grid);
    hipLaunchKernelGGL((k_gemm_mfma_batch<NT, FULL>), dim3((unsigned)grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

template <int NT>
hipError_t run_mfma_batch(const BatchArgs& a, int grid, hipStream_t s) {
    bool full = true;             // as launch_m
    for (int q = 0; q < a.count; ++q) full = full && a.req[q].n >= kSplitKC;
    return full ? run_mfma_batch_f<NT, true>(a, grid, s) : run_mfma_batch_f<NT, false>(a, grid, s);
}

}  // namespace

hipError_t launch_gemm_mfma_batch(const BatchArgs& a, int nt, int grid, hipStream_t s) {
    if (a.count == 0 || a.total_tiles == 0) return hipSuccess;
    hipError_t e;
    switch (nt) {
    case 1: e = run_mfma_batch<1>(a, grid, s); break;
    case 2: e = run_mfma_batch<2>(a, grid, s); break;
    case 4: e = run_mfma_batch<4>(a, grid, s); break;
    case 8: e = run_mfma_batch<8>(a, grid, s); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    return launch_reduce_batch(a, s);
}

// Column-major A, k > 16: one pass over A for all sketch columns (strips of
// kMfmaStrip columns, FP32 partials [S][m][k], FP64 strip sums).  N-tiles per
// workgroup are halved while the launch has fewer tiles than compute units (a
// few-row A, e.g. the n x p factor of the Nystrom second product, where
// generating Omega is the work): each sketch column's sums are the same for
// any N-tile count (the chunk width stays the one of the row-major kernel for
// this k), only A is re-read per column block.
hipError_t launch_gemm_cm_mfma(const CmLaunch& g) {
    const int64_t S = (g.n + kMfmaStrip - 1) / kMfmaStrip;
    const bool skinny = g.m <= 64;
    const int64_t nrb = skinny ? 1 : (g.m + kBM - 1) / kBM;
    int nt = skinny ? 1 : mfma_ntiles(g.k);
    while (!skinny && nt > 1 && S * nrb * ((g.k + 16 * nt - 1) / (16 * nt)) < device_cus()) nt /= 2;
    const int64_t BN = 16 * nt;
    CmMArgs a{};
    a.A = g.A;
    a.m = g.m;
    a.n = g.n;
    a.lda = g.lda;
    a.row0 = g.row0;
    a.key0 = (uint32_t)g.seed;
    a.key1 = (uint32_t)(g.seed >> 32);
    a.col0 = g.col0;
    a.dist = g.dist;
    a.k = g.k;
    a.Y = g.Y;
    a.ldy = g.ldy;
    a.y_trans = g.y_trans;
    a.y_f64 = g.y_f64;
    a.beta = g.beta;
    a.S = (int)S;
    a.partials = a.S > 1 ? static_cast<float*>(g.workspace) : nullptr;
    a.num_rb = (int)nrb;
    a.tiles = (int64_t)a.S * a.num_rb * ((g.k + BN - 1) / BN);
    a.tiles8 = (a.tiles + 7) / 8;
    hipError_t e;
    if (skinny || cm_packed(nt, cm_full(g.n))) {
        // the call's Omega, once (the same plane as the row-major call's); the
        // few-row kernel copies it instead of generating in its workgroups
        PackArgs pk{};
        pk.hi = static_cast<unsigned char*>(g.workspace) + pack_offset(g.m, S, g.k);
        pk.k = g.k;
        pk.kpad = mfma_kpad(g.k);
        pk.key0 = a.key0;
        pk.key1 = a.key1;
        pk.col0 = a.col0;
        pk.dist = a.dist;
        pk.P = 1;
        pk.blk[0] = BlockDesc{g.A, g.n, g.lda, g.row0, nullptr};
        const dim3 pgrid((unsigned)(S * (kMfmaStrip / kSplitKC) / kF32PackChunks),
                         (unsigned)((pk.kpad + kF32PackRows - 1) / kF32PackRows));
        hipLaunchKernelGGL((k_f32_pack<true>), pgrid, dim3(256), 0, g.stream, pk);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        a.fpack = static_cast<const float*>(pk.hi);
        a.kpad = pk.kpad;
    }
    constexpr int KC = kSplitKC;
    if (skinny) {
        const dim3 grid((unsigned)a.tiles), threads(kSkThreads);
        if (g.m % 4 == 0)
            hipLaunchKernelGGL((k_gemm_cm_mfma_skinny<KC, kWhole>), grid, threads, 0, g.stream, a);
        else if (g.m > 4)
            hipLaunchKernelGGL((k_gemm_cm_mfma_skinny<KC, kCut>), grid, threads, 0, g.stream, a);
        else
            hipLaunchKernelGGL((k_gemm_cm_mfma_skinny<KC, kFew>), grid, threads, 0, g.stream, a);
        e = hipGetLastError();
    } else switch (nt) {
    case 1: e = launch_cm_mfma_nt<1, KC>(a, g.stream); break;
    case 2: e = launch_cm_mfma_nt<2, KC>(a, g.stream); break;
    case 4: e = launch_cm_mfma_nt<4, KC>(a, g.stream); break;
    default: e = launch_cm_mfma_nt<8, KC>(a, g.stream); break;
    }
    if (e != hipSuccess || a.S == 1) return e;
    return launch_reduce_partials_t(a.partials, a.S, g.m, g.k, g.Y, g.y_f64, g.ldy, g.beta,
                                    g.y_trans, g.stream);
}

int lp_ntiles(int64_t k) { return k <= 16 ? 1 : k <= 32 ? 2 : 4; }

// Rows per tile of the low-precision kernel: 512 (8 waves of 64 rows share each
// Omega chunk), unless that leaves compute units without a tile, then 256.  Measured on
// 32768^2 with the XCD-grouped tile order: FP8 k = 5 199-201 us against 207-210
// with 256-row tiles, k = 64 299 against 375.  128 and 64 rows (waves of 16) while the
// tiles would fill half the compute units at most, as for the FP32 kernel.
// With 256-row tiles and with these: 5000 x 5000 BF16 k = 64 97 and 52 us, FP8 k = 5 65
// and 47; 2000 x 3000 FP8 k = 64 74 and 36, BF16 k = 16 75 and 54.
static int lp_rows(int64_t m, int64_t strips, int64_t nblk) {
    const auto tiles = [&](int rows) { return strips * ((m + rows - 1) / rows) * nblk; };
    if (tiles(512) >= device_cus()) return 512;
    if (2 * tiles(256) > device_cus()) return 256;
    return 2 * tiles(128) > device_cus() ? 128 : 64;
}

namespace {

int64_t lp_kpad(int64_t k) {
    const int64_t BN = 16 * lp_ntiles(k);
    return (k + BN - 1) / BN * BN;
}

// packed Omega after the partials (pack_offset): hi plane then lo plane,
// strips * kLpStrip * kpad BF16 values each
size_t lp_plane_elems(int64_t strips, int64_t k) {
    return (size_t)strips * (size_t)kLpStrip * (size_t)lp_kpad(k);
}

template <int ADT>
hipError_t launch_lp_pack(const PackArgs& p, int64_t strips, hipStream_t s) {
    const dim3 grid((unsigned)(strips * (kLpStrip / lp_kc(ADT))),
                    (unsigned)((p.kpad + kPackRows - 1) / kPackRows));
    if (p.omega)
        hipLaunchKernelGGL((k_lp_pack<ADT, false>), grid, dim3(256), 0, s, p);
    else
        hipLaunchKernelGGL((k_lp_pack<ADT, true>), grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace

// column-major A: partials, and the packed Omega where a matrix-core kernel
// takes it: the few-row kernel (m <= 64) at every k > 16, the tile kernel at
// k > 32 (whose launch may still run fewer N-tiles and leave it unused)
size_t cm_workspace_bytes(int64_t m, int64_t n, int64_t k) {
    const int64_t S = cm_strips(n, k);
    if (k <= kColGroup) return gemm_workspace_bytes(m, S, k);
    if (m <= 64) return pack_offset(m, S, k) + f32_plane_elems(S, k) * sizeof(float);
    return product_workspace_bytes(0, m, S, k);
}

size_t product_workspace_bytes(int adtype, int64_t m, int64_t strips, int64_t k) {
    if (use_mfma(adtype, k) && mfma_packed(mfma_ntiles(k)))
        return pack_offset(m, strips, k) + f32_plane_elems(strips, k) * sizeof(float);
    if (use_mfma_lp(adtype, k) && lp_packed(lp_ntiles(k)))
        return pack_offset(m, strips, k) + 2 * lp_plane_elems(strips, k) * sizeof(uint16_t);
    return gemm_workspace_bytes(m, strips, k);
}

hipError_t launch_gemm_mfma_lp(const GemmLaunch& g) {
    const int nt = lp_ntiles(g.k);
    const int64_t BN = 16 * nt;
    const int64_t nblk = (g.k + BN - 1) / BN;
    int64_t S = 0;
    for (int b = 0; b < g.P; ++b) S += (g.blk[b].n + kLpStrip - 1) / kLpStrip;
    PackArgs pk{};
    if (lp_packed(nt)) {
        uint16_t* hi = reinterpret_cast<uint16_t*>(static_cast<unsigned char*>(g.workspace) +
                                                   pack_offset(g.m, S, g.k));
        pk.hi = hi;
        pk.lo = hi + lp_plane_elems(S, g.k);
    }
    pk.k = g.k;
    pk.kpad = lp_kpad(g.k);
    pk.key0 = (uint32_t)g.seed;
    pk.key1 = (uint32_t)(g.seed >> 32);
    pk.col0 = g.col0;
    pk.dist = g.dist;
    pk.omega = g.omega;
    pk.ldo = g.ldo;
    pk.P = g.P;
    for (int b = 0; b < g.P; ++b) pk.blk[b] = g.blk[b];
    MArgs a{};
    a.opack = static_cast<const uint16_t*>(pk.hi);
    a.opack_lo = static_cast<const uint16_t*>(pk.lo);
    a.kpad = pk.kpad;
    a.m = g.m;
    a.k = g.k;
    a.ldy = g.ldy;
    a.ldo = g.ldo;
    a.omega = g.omega;
    a.Y = g.Y;
    a.partials = S > 1 ? static_cast<float*>(g.workspace) : nullptr;
    a.key0 = (uint32_t)g.seed;
    a.key1 = (uint32_t)(g.seed >> 32);
    a.col0 = g.col0;
    a.dist = g.dist;
    a.P = g.P;
    a.S_total = (int)S;
    a.y_f64 = g.y_f64;
    a.beta = g.beta;
    for (int b = 0; b < g.P; ++b) a.blk[b] = g.blk[b];
    const int rows = lp_rows(g.m, S, nblk);
    a.nblk = (int)nblk;
    const TraceEvents& tr = g.trace;
    if (tr.begin) (void)hipEventRecord(tr.begin, g.stream);
    hipError_t e = hipSuccess;
    if (lp_packed(nt)) {
        e = g.adtype == 1 ? launch_lp_pack<1>(pk, S, g.stream) : launch_lp_pack<2>(pk, S, g.stream);
        if (e != hipSuccess) return e;
    }
    const bool gen = (g.omega == nullptr);
    e = g.adtype == 1 ? dispatch_lp<1>(nt, gen, rows, a, g.stream)
                      : dispatch_lp<2>(nt, gen, rows, a, g.stream);
    if (e != hipSuccess) return e;
    if (tr.mid) (void)hipEventRecord(tr.mid, g.stream);
    if (S > 1) e = launch_reduce_partials(a.partials, (int)S, g.m, g.k, g.Y, g.y_f64, g.ldy,
                                          g.beta, g.stream);
    if (tr.end) (void)hipEventRecord(tr.end, g.stream);
    return e;
}

namespace {

template <int NT, int ADT>
hipError_t run_lp_batch(const BatchArgs& a, int grid, hipStream_t s) {
    static const int per_cu = [] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_gemm_mfma_lp_batch<NT, ADT>,
                                                         64 * kLpBatchWaves, 0) != hipSuccess)
            n = 1;
        return n;
    }();
    grid = batch_grid(per_cu, a.total_tiles, grid);
    hipLaunchKernelGGL((k_gemm_mfma_lp_batch<NT, ADT>), dim3((unsigned)grid),
                       dim3(64 * kLpBatchWaves), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_mfma_lp_batch(const BatchArgs& a, int nt, int adtype, int grid,
                                     hipStream_t s) {
    if (a.count == 0 || a.total_tiles == 0) return hipSuccess;
    hipError_t e;
    if (adtype == 1) {
        e = nt == 1 ? run_lp_batch<1, 1>(a, grid, s) : nt == 2 ? run_lp_batch<2, 1>(a, grid, s)
                                                              : run_lp_batch<4, 1>(a, grid, s);
    } else {
        e = nt == 1 ? run_lp_batch<1, 2>(a, grid, s) : nt == 2 ? run_lp_batch<2, 2>(a, grid, s)
                                                              : run_lp_batch<4, 2>(a, grid, s);
    }
    if (e != hipSuccess) return e;
    return launch_reduce_batch(a, s);
}

}  // namespace sk
