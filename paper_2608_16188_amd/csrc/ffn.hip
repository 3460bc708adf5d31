// Expert MLP forward and backward as grouped GEMMs on gfx950.
//
// bf16 path: one templated matrix-core kernel, C[M x N] = sum_k A(m,k) B(n,k),
// one output tile of one expert per block. The tiles of nearly every launch
// are 256 x 256 or 256 x 192 (PhaseTile<>, phase_tile: eight waves, one block
// per CU, 64-deep stages taken in 64-column phases); small weight gradients
// take 128 x 128 with four waves on a plain ring of stages (SmallTile, ring_tile,
// two blocks per CU); a few rows an expert take small_rows_kernel forward. A wave
// accumulates its sub-tile with v_mfma_f32_32x32x16_bf16 in f32. Operands reach LDS through buffer loads that write LDS directly (16
// bytes per lane, out-of-range offsets read as zero, so ragged tails need no
// branch); later stages' loads stay in flight across the barriers (partial
// vmcnt waits).
// An operand whose k index is contiguous in HBM is stored k-major with an
// XOR chunk swizzle; one whose k index is strided (weights read transposed
// in the backward, the token-reduced weight-gradient GEMMs) is copied
// unchanged, mn-major, and its fragments are read with ds_read_b64_tr_b16.
// The operand roles are swapped inside the MFMA so each lane holds runs of
// consecutive output columns of one row; the fused epilogues (bias, GELU and
// GELU' pair, GELU' product, bf16 rounding, f32 weight gradients with the
// bias-gradient row sums) park the tile in LDS and store 16-byte row
// segments.
//
// Each expert's row count n_e = sum_g counts[g, e] is read on the device:
// tiles past n_e exit at once (M = n_e GEMMs) or n_e bounds the k loop
// (weight-gradient GEMMs, which still write zeros for an empty expert).
// Blocks are mapped so that each XCD works on a contiguous run of tiles,
// grouped group_m m-tiles at a time, which keeps operand panels in that
// XCD's L2. The tile shape is chosen per launch by a cost model: rounds of
// 256 CUs times the tile area, scaled by a per-shape efficiency.
//
// f32 path: 32 x 32 or 64 x 64 tiles on the f32 matrix cores
// (v_mfma_f32_32x32x2f32), four waves splitting k, with the same operand and
// epilogue description (the accuracy path).
#include <mutex>
#include <type_traits>

#include "common.h"

namespace vmoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

enum Epi { EPI_FWD1 = 0, EPI_BIAS = 1, EPI_GELU_GRAD = 2, EPI_STORE = 3, EPI_F32 = 4 };

// Operand: element (mn, k) of expert e is
//   k-major : base[e*estride + mn*ld + k]
//   mn-major: base[e*estride + k*ld + mn]
struct Operand {
    const void* base;
    long long estride;
    int ld;
};

struct GemmArgs {
    Operand a, b;
    int M, N, K;            // static sizes; M or K is replaced by n_e (see var_k)
    int var_k;              // 0: M = n_e, 1: K = n_e
    const int32_t* counts;  // [G, E]
    int G, E;
    void* out;              // primary output (EPI_FWD1: gelu(H))
    void* out2;             // EPI_FWD1: gelu'(H)
    long long out_estride;
    int ldo;
    const void* bias;       // EPI_FWD1 / EPI_BIAS
    long long bias_estride;
    const void* aux;        // EPI_GELU_GRAD: saved gelu'(H)
    float* bsum;            // EPI_F32: row sums of A per expert, or null
    // Gathered operand (kernels built with GATHER != 0): the operand's rows
    // are token rows of x, row r of expert e being x[tok[e * tok_estride + r]];
    // its base is x itself (estride 0) and gather_bytes the size of x.
    const int32_t* tok;     // null: this problem's operand is not gathered
    long long tok_estride;
    long long gather_bytes;
};


// Up to two independent GEMMs of one kernel instantiation in one launch (the
// two weight gradients): blocks [0, total[0]) work on problem 0, the rest on
// problem 1, so the second fills the first's last, partial round of tiles.
struct GemmBatch {
    GemmArgs p[2];
    int tiles_m[2], tiles_n[2], total[2];
    int group_m, chunk, per_xcd;
};

// A GEMM whose m is the expert's rows (every epilogue but the weight
// gradients', whose k is the rows) runs one problem per launch and numbers its
// tiles over the experts' live m-tiles only (ceil(n_e / BM) each, from the
// device row counts): the blocks past the last live tile all sit at the end
// of the grid instead of between the live tiles of consecutive experts, where
// each would hold a CU slot while the dispatcher places blocks in order.
template <int EPI>
constexpr bool compact_tiles() { return EPI != EPI_F32; }

// Rows of expert e: sum over the groups, sixteen counts in flight at a time (a
// single group's count is one load: sixteen of the same word at the head of every
// tile cost the one-group ViT-L/16 step 1064 -> 1050 us, one image 50.6 -> 50.0).
__device__ __forceinline__ int expert_rows(const int32_t* counts, int G, int E, int e) {
    constexpr int U = 16;
    if (G == 1) return counts[e];
    int n = 0;
    for (int g0 = 0; g0 < G; g0 += U) {
        int v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = counts[min(g0 + u, G - 1) * E + e];
#pragma unroll
        for (int u = 0; u < U; ++u) n += g0 + u < G ? v[u] : 0;
    }
    return n;
}

// Inclusive sum over the lanes of a wave, in DPP adds (a few cycles each; the
// six dependent LDS shuffles of the usual form are most of a microsecond, at
// the start of every tile).
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15, rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31, rows 2, 3
    return v;
}

// m-tiles of an expert with ne rows: ceil(ne / bm), except that an expert
// whose rows fit one 32-row block (a light expert) gets `lsplit` tiles per
// n-tile, each taking a share of the tile's columns (its weight stream then
// runs on lsplit CUs). lsplit = 1 leaves every expert at ceil(ne / bm).
__device__ __forceinline__ int expert_mtiles(int ne, int bm, int lsplit) {
    return lsplit > 1 && ne > 0 && ne <= 32 ? lsplit : (ne + bm - 1) / bm;
}

// Live tile w of a compact problem: lane e of every wave sums expert e's rows
// (at most `cap`, the rows of its buffer) and its tile count, an inclusive
// scan over the lanes places the experts' tile ranges end to end, and the
// expert holding w is the number of ranges that end at or before it. Returns
// false past the last live tile. Uniform per wave (every wave of a block
// computes the same).
struct LiveTile {
    int e, r, ne;  // expert, tile index inside the expert, expert's rows
};
__device__ __forceinline__ bool live_tile(const int32_t* counts, int G, int E, int cap, int bm,
                                          int lsplit, int tiles_n, int w, LiveTile* out) {
    const int lane = threadIdx.x & 63;
    // (never past the expert's rows, whatever the counts say)
    const int ne = lane < E ? min(expert_rows(counts, G, E, lane), cap) : 0;
    const int t = expert_mtiles(ne, bm, lsplit) * tiles_n;
    const int incl = wave_scan(t);
    if (w >= __builtin_amdgcn_readlane(incl, 63)) return false;
    const int e = __popcll(__ballot(incl <= w));
    out->e = e;
    out->r = w - __builtin_amdgcn_readlane(incl - t, e);
    out->ne = __builtin_amdgcn_readlane(ne, e);
    return true;
}

// Row GEMMs whose outputs are d wide, under a skewed load. The launch order
// is cut into chunks of `chunk` tiles; a chunk runs on one XCD (chunks are
// dealt to the XCDs in turn) and its tiles share operand panels in that
// XCD's L2. With lsplit = 1 (light tiles as long as a heavy one's weight
// stream) the chunks of heavy experts' live tiles (at least half a tile of
// rows) are spread evenly over the first 70% of the chunk positions and those
// of light experts fill the rest, so that light tiles do not run alone at the
// end. Inside each class experts go in order; with no light expert it is the
// plain live-tile order. Measured at the ViT-L/16 skew (four full experts, 28
// of ~17 rows): the spread took the down-projection 216 -> 178 us and dxe
// 204 -> 161 us against expert order (few n-tiles, long k); it slowed the
// f-wide row GEMMs (196 -> 213, 173 -> 191 us) and the weight gradients
// (350 -> 399: heavy tiles apart no longer shared panels in L2), which keep
// the plain order. With lsplit > 1 (light tiles split into short column
// parts) every XCD instead takes an equal contiguous share of the heavy
// tiles first, all of them starting in the first round, then an equal
// contiguous share of the light parts, which run on its remaining CUs beside
// them: x is the block's XCD, c its place in that XCD's block sequence (i is
// unused). Chunk position c, tile i inside it (lsplit = 1); false past the
// class's tiles. Uniform per wave.
__device__ __forceinline__ bool spread_tile(const GemmBatch& batch, int bm, int lsplit, int x,
                                            int c, int i, int* e_out, int* r_out, int* ne_out) {
    const GemmArgs& p0 = batch.p[0];
    const int E = p0.E, lane = threadIdx.x & 63, chunk = batch.chunk;
    int ne = 0;
    if (lane < E) ne = min(expert_rows(p0.counts, p0.G, E, lane), p0.M);
    const bool heavy_l = lane < E && 2 * ne >= bm;
    const int te = lane < E ? expert_mtiles(ne, bm, lsplit) * batch.tiles_n[0] : 0;
    // either class's experts' tile ranges end to end (inclusive scans)
    const int th = heavy_l ? te : 0, tl = te - th;
    const int ih = wave_scan(th), il = wave_scan(tl);
    const int nh = __builtin_amdgcn_readlane(ih, 63), nl = __builtin_amdgcn_readlane(il, 63);
    bool heavy;
    int j;  // index in the class's list
    if (lsplit > 1) {
        const int h0 = x * nh / 8, hx = (x + 1) * nh / 8 - h0;
        heavy = c < hx;
        j = heavy ? h0 + c : x * nl / 8 + (c - hx);
        if (!heavy && c - hx >= (x + 1) * nl / 8 - x * nl / 8) return false;
    } else {
        const int nhc = (nh + chunk - 1) / chunk, nlc = (nl + chunk - 1) / chunk;
        const int first = max(nhc, (7 * (nhc + nlc) + 9) / 10);
        int ci;
        if (c < first) {
            const int hc = static_cast<int>((static_cast<long long>(c) + 1) * nhc / first);
            const int hp = static_cast<int>(static_cast<long long>(c) * nhc / first);
            heavy = hc > hp;
            ci = heavy ? hp : c - hc;
        } else {
            heavy = false;
            ci = c - nhc;
        }
        j = ci * chunk + i;
    }
    if (j >= (heavy ? nh : nl)) return false;
    const int t = heavy ? th : tl, incl = heavy ? ih : il;
    const int e = __popcll(__ballot(incl <= j));
    *e_out = e;
    *r_out = j - __builtin_amdgcn_readlane(incl - t, e);
    *ne_out = __builtin_amdgcn_readlane(ne, e);
    return true;
}

// ------------------------------------------------------------------ quotas

// Fill-clamp-refill (the paper's lifespan aligning, Sec. 3.2.2) on one wave,
// lane i holding expert i (n <= 64): every expert starts from its minimum,
// the budget left is split among the unsaturated experts in proportion to
// their coefficients, an expert pushed past its saturation is clamped and
// its excess shared again, until nothing is returned; then the real shares
// are rounded to floor(sum) whole units by largest remainder (ties to the
// lower index). Every sum runs in ascending expert order with the host
// routine's operations (vmoe_fill_clamp_refill), so the units equal its
// units for the same inputs. Returns lane i's units (0 past n).
__device__ int fill_clamp_refill_wave(int n, int mn, int sat, double coef, int budget) {
    const int lane = threadIdx.x & 63;
    const bool valid = lane < n;
    double a = valid ? static_cast<double>(mn) : 0.0;
    long long need = 0;
    for (int r = 0; r < n; ++r) need += __shfl(mn, r, 64);
    bool act = valid && a < static_cast<double>(sat) && coef > 0.0;
    double left = static_cast<double>(budget - need);
    while (left > 0.0 && __ballot(act) != 0ull) {
        double W = 0.0;
        for (int r = 0; r < n; ++r) {
            const double c = __shfl(coef, r, 64);
            if (__shfl(static_cast<int>(act), r, 64)) W += c;
        }
        if (act) a += left * coef / W;
        left = 0.0;
        for (int r = 0; r < n; ++r) {
            const double ar = __shfl(a, r, 64);
            const int sr = __shfl(sat, r, 64);
            if (__shfl(static_cast<int>(act), r, 64) && ar > static_cast<double>(sr))
                left += ar - static_cast<double>(sr);
        }
        if (act && a > static_cast<double>(sat)) {
            a = static_cast<double>(sat);
            act = false;
        }
    }
    const double fl = floor(a);
    int units = static_cast<int>(fl);
    long long base = 0;
    double sum = 0.0;
    for (int r = 0; r < n; ++r) {
        base += __shfl(units, r, 64);
        sum += __shfl(a, r, 64);
    }
    long long extra = static_cast<long long>(floor(sum + 1e-9)) - base;
    bool up = false;  // rounded up already
    while (extra > 0) {
        // the largest fractional part not yet rounded up, lowest index on ties
        const double fr = (valid && !up) ? a - fl : 0.0;
        int best = -1;
        double bf = 0.0;
        for (int r = 0; r < n; ++r) {
            const double f = __shfl(fr, r, 64);
            if (f > bf) {
                best = r;
                bf = f;
            }
        }
        if (best < 0) break;
        if (lane == best) {
            ++units;
            up = true;
        }
        --extra;
    }
    return valid ? units : 0;
}

// The quota plan of one launch: per expert its rows, its tiles, the first of
// its blocks and the number of blocks it gets.
struct QuotaPlan {
    int ne[64], tiles[64], first[64], units[64];
};

// Work model of one expert's tiles, in relative time units: a tile of the
// GEMMs whose m is the expert's rows costs a fixed part (streaming its
// weight panel) plus a part in proportion to its live rows; a weight-gradient
// tile a fixed part (its output writes) plus one in proportion to the rows it
// reduces over (300 rows ~ the writes of a 256-column tile, as measured).
template <int EPI>
__device__ __forceinline__ double tile_work(int ne, int bm) {
    if constexpr (EPI == EPI_F32) return static_cast<double>(ne) + 300.0;
    else return 1.0 + static_cast<double>(min(ne, bm)) / bm;
}

constexpr bool compact_epi(int epi) { return epi != EPI_F32; }

// Wave 0 forms the launch's plan: per expert its rows and tiles, its work
// (tiles x tile_work) as the coefficient, its tiles as saturation, a minimum
// of one block when it has tiles, and the fill-clamp-refill split of the
// launch's blocks; experts own consecutive block ranges in expert order.
template <int EPI>
__device__ void build_quota_plan(const GemmBatch& batch, int bm, int lsplit, int budget,
                                 QuotaPlan* qp) {
    const int lane = threadIdx.x & 63;
    const GemmArgs& p0 = batch.p[0];
    const int E = p0.E;
    int ne = 0;
    if (lane < E)
        for (int g = 0; g < p0.G; ++g) ne += p0.counts[g * E + lane];
    int tiles = 0;
    if (lane < E) {
        if constexpr (compact_epi(EPI)) {
            ne = min(ne, p0.M);
            tiles = expert_mtiles(ne, bm, lsplit) * batch.tiles_n[0];
        } else {
            tiles = batch.tiles_m[0] * batch.tiles_n[0] +
                    (batch.total[1] > 0 ? batch.tiles_m[1] * batch.tiles_n[1] : 0);
        }
    }
    // (a light expert's column parts each carry a share of one tile's stream)
    const bool parts = lsplit > 1 && ne > 0 && ne <= 32;
    const double coef = static_cast<double>(tiles) * tile_work<EPI>(ne, bm) / (parts ? lsplit : 1);
    const int units = fill_clamp_refill_wave(E, tiles > 0 ? 1 : 0, tiles, coef, budget);
    int incl = units;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    qp->ne[lane] = ne;
    qp->tiles[lane] = tiles;
    qp->first[lane] = incl - units;
    qp->units[lane] = units;
}

__device__ __forceinline__ float gelu_f(float h) {
    return 0.5f * h * (1.0f + erff(h * 0.70710678118654752f));
}

__device__ __forceinline__ float gelu_grad_f(float h) {
    return 0.5f * (1.0f + erff(h * 0.70710678118654752f)) +
           h * 0.39894228040143268f * __expf(-0.5f * h * h);
}

// ------------------------------------------------------------------ bf16 MFMA

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// The wave's index in its block, as a scalar.
__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
}

// Operand stages of KB k values (32 or 64) in LDS, filled by buffer_load ... lds:
// lane L of a wave instruction fills bytes [16 L, 16 L + 16) of a 1 KB block, so
// rows are unpadded and 16-byte chunks are XOR-swizzled instead (k-major: chunk ^
// ((row / P) mod Q) with P rows per 256 bytes and Q chunks per row; mn-major: chunk
// ^ s (k mod 4) with s = 4, or 2 when a row's chunk count is a multiple of 8 but
// not 16, so the XOR stays inside the row), which keeps fragment and transpose
// reads free of bank conflicts.

// XOR applied to the 16-byte chunk index of k-row k of an mn-major DMA stage.
template <int ROWS>
__device__ __forceinline__ int mn_swizzle(int k) {
    static_assert((ROWS / 8) % 8 == 0, "mn-major rows must hold a multiple of 8 chunks");
    constexpr int SHIFT = (ROWS / 8) % 16 == 0 ? 2 : 1;
    return (k & 3) << SHIFT;
}

// Element offset (in bf16) of (mn, k) inside one operand stage.
template <int ROWS, bool KMAJOR, int KB>
__device__ __forceinline__ int lds_off(int mn, int k) {
    if constexpr (KMAJOR) {
        constexpr int Q = KB / 8, P = 16 / Q;  // chunks per row, rows per 256 bytes
        return mn * KB + (((k >> 3) ^ ((mn / P) % Q)) << 3) + (k & 7);
    } else {
        return k * ROWS + (((mn >> 3) ^ mn_swizzle<ROWS>(k)) << 3) + (mn & 7);
    }
}

// Byte offset in HBM of the 16-byte vector holding (mn, k..k+7) [k-major] or
// (k, mn..mn+7) [mn-major], or kOutOfRange when it lies outside the operand.
template <bool KMAJOR>
__device__ __forceinline__ uint32_t vec_off(int ld, int mn, int mn_lim, int k, int k_lim) {
    const bool ok = (mn < mn_lim) && (k < k_lim);
    const int e = KMAJOR ? mn * ld + k : k * ld + mn;
    return ok ? static_cast<uint32_t>(e) * 2u : kOutOfRange;
}

// An operand stage is ROWS * KB / 512 blocks of 1 KB; wave w
// issues blocks [w * PER, (w + 1) * PER). Lane L of a block holds physical
// bytes [16 L, 16 L + 16), whose logical (swizzled) position decides what it
// fetches.
template <int ROWS, bool KMAJOR, int KB, int NT>
struct DmaStage {
    static constexpr int BLOCKS = ROWS * KB * 2 / 1024;
    static constexpr int PER = BLOCKS / (NT / 64);  // wave instructions per stage
    static_assert(PER >= 1 && PER * (NT / 64) == BLOCKS, "1 KB blocks must split evenly over waves");
    static __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, int ld, int mn0,
                                                 int mn_lim, int k0, int k_lim, uint16_t* s) {
        const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int blk = wave * PER + q;
            const int byte = blk * 1024 + 16 * lane;
            uint32_t off;
            if (KMAJOR) {
                constexpr int RB = KB * 2, Q = KB / 8, P = 16 / Q;
                const int r = byte / RB;
                const int c = ((byte % RB) >> 4) ^ ((r / P) % Q);
                off = vec_off<true>(ld, mn0 + r, mn_lim, k0 + 8 * c, k_lim);
            } else {
                constexpr int RB = ROWS * 2;  // bytes per k row
                const int r = byte / RB;
                const int c = ((byte % RB) >> 4) ^ mn_swizzle<ROWS>(r);
                off = vec_off<false>(ld, mn0 + 8 * c, mn_lim, k0 + r, k_lim);
            }
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void*)(s + blk * 512), 16, off, 0, 0, 0);
        }
    }
    // Stages that lie inside K: the lane's byte offset of wave instruction q at
    // k = 0 (kOutOfRange outside the operand) holds for every stage, whose k
    // goes into the scalar offset, so a stage costs its PER instructions and
    // no per-lane arithmetic.
    static __device__ __forceinline__ void lane_offs(int ld, int mn0, int mn_lim,
                                                     uint32_t (&off)[PER]) {
        const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int byte = (wave * PER + q) * 1024 + 16 * lane;
            if (KMAJOR) {
                constexpr int RB = KB * 2, Q = KB / 8, P = 16 / Q;
                const int r = byte / RB;
                const int c = ((byte % RB) >> 4) ^ ((r / P) % Q);
                off[q] = vec_off<true>(ld, mn0 + r, mn_lim, 8 * c, KB);
            } else {
                constexpr int RB = ROWS * 2;
                const int r = byte / RB;
                const int c = ((byte % RB) >> 4) ^ mn_swizzle<ROWS>(r);
                off[q] = vec_off<false>(ld, mn0 + 8 * c, mn_lim, r, KB);
            }
        }
    }
    // (k-major, gathered rows: rowoff as in issue_rows)
    static __device__ __forceinline__ void lane_offs_rows(const int (&rowoff)[PER],
                                                          uint32_t (&off)[PER]) {
        static_assert(KMAJOR, "row gather: k-major operand");
        const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int byte = (wave * PER + q) * 1024 + 16 * lane;
            constexpr int RB = KB * 2, Q = KB / 8, P = 16 / Q;
            const int c = ((byte % RB) >> 4) ^ ((byte / RB / P) % Q);
            off[q] = rowoff[q] >= 0 ? static_cast<uint32_t>(rowoff[q] + 8 * c) * 2u : kOutOfRange;
        }
    }
    static __device__ __forceinline__ void issue_inside(__amdgpu_buffer_rsrc_t rs,
                                                        const uint32_t (&off)[PER],
                                                        uint32_t k_bytes, uint16_t* s) {
        const int wave = wave_id();
#pragma unroll
        for (int q = 0; q < PER; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void*)(s + (wave * PER + q) * 512), 16,
                off[q], k_bytes, 0, 0);
    }
    // Gathered operands (rows of x): the stage row lane L fetches in wave
    // instruction q (k-major: an mn row of the tile; mn-major: a k row).
    static __device__ __forceinline__ int lane_row(int q) {
        const int lane = threadIdx.x & 63, wave = wave_id();
        const int byte = (wave * PER + q) * 1024 + 16 * lane;
        return byte / (KMAJOR ? KB * 2 : ROWS * 2);
    }
    // k-major, gathered rows: rowoff[q] = element offset in x of the start of
    // the row lane_row(q) stands for (-1 past the rows).
    static __device__ __forceinline__ void issue_rows(__amdgpu_buffer_rsrc_t rs,
                                                      const int (&rowoff)[PER], int k0,
                                                      int k_lim, uint16_t* s) {
        static_assert(KMAJOR, "row gather: k-major operand");
        const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int blk = wave * PER + q;
            const int byte = blk * 1024 + 16 * lane;
            constexpr int RB = KB * 2, Q = KB / 8, P = 16 / Q;
            const int r = byte / RB;
            const int c = ((byte % RB) >> 4) ^ ((r / P) % Q);
            const int kk = k0 + 8 * c;
            const uint32_t off = (rowoff[q] >= 0 && kk < k_lim)
                                     ? static_cast<uint32_t>(rowoff[q] + kk) * 2u
                                     : kOutOfRange;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void*)(s + blk * 512), 16, off, 0, 0, 0);
        }
    }
    // mn-major, gathered k rows: rowoff[q] = byte offset in x of the k row
    // lane_row(q) stands for in this stage, col[q] = byte offset of the lane's
    // 8 columns in it (krow_cols); either is kGatherSentinel outside the
    // operand, which puts the sum past the end of x.
    static __device__ __forceinline__ void krow_cols(int mn0, int mn_lim, uint32_t (&col)[PER]) {
        static_assert(!KMAJOR, "k-row gather: mn-major operand");
        const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int byte = (wave * PER + q) * 1024 + 16 * lane;
            constexpr int RB = ROWS * 2;
            const int r = byte / RB;
            const int mn = mn0 + 8 * (((byte % RB) >> 4) ^ mn_swizzle<ROWS>(r));
            col[q] = mn < mn_lim ? static_cast<uint32_t>(mn) * 2u : kGatherSentinel;
        }
    }
    static __device__ __forceinline__ void issue_krows(__amdgpu_buffer_rsrc_t rs,
                                                       const uint32_t (&rowoff)[PER],
                                                       const uint32_t (&col)[PER], uint16_t* s) {
        const int wave = wave_id();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int blk = wave * PER + q;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void*)(s + blk * 512), 16,
                rowoff[q] + col[q], 0, 0, 0);
        }
    }
};

// s_waitcnt immediate for vmcnt(n) and lgkmcnt(0) (expcnt left alone).
template <int N>
struct VmWait {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    static constexpr int imm = (N & 15) | ((N >> 4) << 14) | (7 << 4);
};

// Workgroup barrier for the operand stages. __syncthreads() fences all memory at
// workgroup scope, which waits for every LDS DMA in flight (vmcnt(0)) and
// would cap the prefetch at one stage, so the callers see to two things
// themselves: the DMA of what is read next has landed (their s_waitcnt on vmcnt),
// and this wave's reads of what is refilled next are done. The ring of whole
// stages waits for the latter too (lgkmcnt(0) in VmWait). phase_tile does not: it
// refills a panel, or a stage's A, one phase after the phase whose products
// consumed the fragments read from it, and consuming them waited for those reads.
// The signal fences keep the compiler from moving memory accesses across it.
__device__ __forceinline__ void ring_barrier() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// A barrier that waits for this wave's LDS accesses only: its stores stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// ds_read_b64_tr_b16: within each 16-lane group, lane j reads 4 bf16 at its
// address and lane i receives element i % 4 of lanes i/4, i/4+4, i/4+8, i/4+12.
// With lane j pointing at row j/4, column 4*(j%4) of a 4 x 16 block, lane i
// gets column i: four consecutive k values of one mn index.
__device__ __forceinline__ s16x4 lds_read_tr(const uint16_t* p) {
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p));
}

// Operand fragment of v_mfma_f32_32x32x16_bf16 for 32 mn values (lane & 31)
// x 8 k values (k = 16 * kstep + 8 * (lane >> 5) + 0..7).
template <int ROWS, bool KMAJOR, int KB>
__device__ __forceinline__ bf16x8 read_frag(const uint16_t* s, int blk, int kstep, int lane) {
    if (KMAJOR) {
        const int mn = blk * 32 + (lane & 31), k = kstep * 16 + (lane >> 5) * 8;
        return *reinterpret_cast<const bf16x8*>(s + lds_off<ROWS, true, KB>(mn, k));
    } else {
        // 16-lane group g covers mn [16 (g & 1), +16) and k [8 (g >> 1), +8)
        const int g = lane >> 4, j = lane & 15;
        const int k = kstep * 16 + 8 * (g >> 1) + (j >> 2);
        const int mn = blk * 32 + 16 * (g & 1) + 4 * (j & 3);
        const s16x4 lo = lds_read_tr(s + lds_off<ROWS, false, KB>(mn, k));
        const s16x4 hi = lds_read_tr(s + lds_off<ROWS, false, KB>(mn, k + 4));
        const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, v);
    }
}

// GELU and its derivative from one exponential. With phi the standard normal
// density, Abramowitz & Stegun 26.2.17 gives the upper tail
//   q = 1 - Phi(|h|) = phi(h) t (b1 + t (b2 + t (b3 + t (b4 + t b5)))),
//   t = 1 / (1 + p |h|), |error| < 7.5e-8 (far below bf16 rounding), so
//   Phi(h) = 0.5 + sign(h) (0.5 - q),  gelu(h) = h Phi(h),  gelu'(h) = Phi(h) + h phi(h),
// where phi(h) = 2^(-h^2 log2(e) / 2 + log2(1 / sqrt(2 pi))) is one v_exp_f32.
__device__ __forceinline__ void gelu_pair(float h, float& g, float& dg) {
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(fabsf(h), 0.2316419f, 1.0f));
    const float phi = __builtin_amdgcn_exp2f(
        __builtin_fmaf(h * h, -0.72134752044448170f, -1.32574806473615920f));
    float poly = __builtin_fmaf(t, 1.330274429f, -1.821255978f);
    poly = __builtin_fmaf(t, poly, 1.781477937f);
    poly = __builtin_fmaf(t, poly, -0.356563782f);
    poly = __builtin_fmaf(t, poly, 0.319381530f);
    const float q = (t * poly) * phi;
    const float phi_cdf = 0.5f + copysignf(0.5f - q, h);
    g = h * phi_cdf;
    dg = __builtin_fmaf(h, phi, phi_cdf);
}

// The 128 x 128 tile of small weight gradients: four waves as 2 x 2, a ring of four
// 32-deep stages, two blocks per CU.
struct SmallTile {
    static constexpr int BM = 128, BN = 128, WGN = 2, KB = 32, NS = 4;
    static constexpr bool PHASED = false;
    static constexpr int NW = 4, NT = 256, WAVES_PER_EU = 2;
    static constexpr int WM = 64, WN = 64, FM = 2, FN = 2;  // wave tile, in 32 x 32 blocks
    static constexpr int KSTEPS = KB / 16;
    static constexpr int RING_BYTES = NS * (BM + BN) * KB * 2;
};

// A 256-row tile whose 64-deep stages are worked through in PB phases, one per
// 64-column panel of B (phase_tile below): eight waves as 4 x 2, a wave's 64
// rows against 32 columns of the phase's panel.
template <int PB_>
struct PhaseTile {
    static constexpr int PB = PB_;
    static constexpr int BM = 256, BN = 64 * PB, WGN = 2, KB = 64, NS = 2;
    static constexpr bool PHASED = true;
    static constexpr int NW = 8, NT = 512, WAVES_PER_EU = 2;
    static constexpr int WM = 64, FM = 2;
    // LDS: two A stages, two stages of PB panels of B (panels 0, 1 and the rest
    // in arrays of their own, so that the compiler can tell a read of one from
    // the loads in flight into another), the epilogue's 4 KB a wave
    static constexpr int A_EL = BM * KB, P_EL = 64 * KB, S_EL = NW * 2048;
    static constexpr int BL_EL = 2 * P_EL, BH_EL = (PB - 2) * P_EL;
};

// The shape a phased kernel's light tiles use (light_tile): 64-column wave
// columns and one 32-row block, each wave's LDS in a 16 KB buffer of its own.
template <int COLS>
struct LightShape {
    static constexpr int BM = 32, BN = 64 * COLS, WGN = COLS, NS = 8, NW = 8, NT = 512;
    static constexpr int WM = 32, WN = 64, FM = 1, FN = 2;
    static constexpr int RING_BYTES = NS * 16384;
    static constexpr bool PHASED = false;
};

// Static sizes of gemm_epilogue, for small and light tiles: wave w parks one 32-row
// block of its outputs, all outputs at once, in 16 KB buffer w. Staged rows are
// padded by 16 bytes: 16-byte aligned for the row reads (a 136-byte bf16 row left
// every other row's reads misaligned, which the LDS serves with stalls) and off the
// banks of the row above.
template <class T, int EPI>
struct GemmCfg {
    static constexpr int BUF_BYTES = T::RING_BYTES / T::NS;  // one stage buffer
    static constexpr bool F32_OUT = EPI == EPI_F32;
    static constexpr int OUTS = EPI == EPI_FWD1 ? 2 : 1;
    static constexpr int ELEM = F32_OUT ? 4 : 2;
    static constexpr int EP_LD = T::WN + 16 / ELEM;
    static constexpr int EP_TILE = 32 * EP_LD * ELEM;
    static_assert(T::NW <= T::NS && OUTS * EP_TILE <= BUF_BYTES, "epilogue staging exceeds LDS");
    static_assert(!F32_OUT || T::NT % T::BM == 0, "row sums give each A row NT / BM threads");
    static_assert(!F32_OUT || T::NT * 4 <= BUF_BYTES, "row-sum partials fit one stage buffer");
};

template <class T>
struct Frags {
    static constexpr int FM = T::FM, FN = T::FN;
    bf16x8 a[FM], b[FN];
    // FL: the wave's first FL 32-row blocks are read (0: none, and no B either)
    template <int FL>
    __device__ __forceinline__ void read(const uint16_t* As, const uint16_t* Bs, int wm, int wn,
                                         int ks, int lane) {
        if constexpr (FL > 0) {
#pragma unroll
            for (int i = 0; i < FL; ++i)
                a[i] = read_frag<T::BM, false, T::KB>(As, wm * FM + i, ks, lane);
#pragma unroll
            for (int j = 0; j < FN; ++j)
                b[j] = read_frag<T::BN, false, T::KB>(Bs, wn * FN + j, ks, lane);
        }
    }
};

// acc[i][j] += A-block i x B-block j for the row blocks i < FL; the operands
// are swapped inside the MFMA so that register 4q + r of lane l holds
// C[m = l % 32][n = 8q + 4 (l / 32) + r].
template <int FL, int FM, int FN, typename F>
__device__ __forceinline__ void mfma_block(f32x16 (&acc)[FM][FN], const F& f) {
#pragma unroll
    for (int i = 0; i < FL; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
}

// Bias of the columns a lane owns: column 32 j + 8 q + 4 (l / 32) + 0..3 of the
// wave tile, for j < FN, q < 4, as four packed bf16 (zero past N). Loaded ahead
// of the first operand stages; the accumulators start from it.
template <class T, int EPI>
struct BiasRegs {
    static constexpr bool USED = EPI == EPI_FWD1 || EPI == EPI_BIAS;
    uint2 v[USED ? T::FN * 4 : 1];
    __device__ __forceinline__ void load(const GemmArgs& p, int e, int N, int n0, int wn, int lane) {
        if constexpr (USED) {
#pragma unroll
            for (int j = 0; j < T::FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = n0 + wn * T::WN + j * 32 + 8 * q + 4 * (lane >> 5);
                    v[j * 4 + q] = n < N ? *reinterpret_cast<const uint2*>(
                                               static_cast<const uint16_t*>(p.bias) +
                                               e * p.bias_estride + n)
                                         : make_uint2(0u, 0u);
                }
        }
    }
};

// Epilogue of one block: optional bias-gradient row sums (partials combined in
// part_buf), then each wave turns its accumulators (bias included) into outputs (GELU +
// GELU', GELU' product), parks them in its own slot of ep_buf and writes every
// output row as 16-byte-per-lane segments. The slots are private to a wave and
// LDS accesses of one wave complete in order, so the passes need no barrier.
template <class T, class CFG, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& p, f32x16 (&acc)[T::FM][T::FN],
                                              uint16_t* part_buf,
                                              uint16_t* ep_buf, float rsum, bool row_sum, int e,
                                              int M, int N, int m0, int n0, int fm_live) {
    constexpr int FM = T::FM, FN = T::FN, WM = T::WM, WN = T::WN, BM_ = T::BM;
    constexpr int EP_LD = CFG::EP_LD, ELEM = CFG::ELEM, EP_TILE = CFG::EP_TILE;
    constexpr int OUTS = CFG::OUTS;
    constexpr bool F32_OUT = CFG::F32_OUT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / T::WGN, wn = wave % T::WGN;

    if constexpr (F32_OUT) {
        if (row_sum) {  // uniform per block
            constexpr int SPLIT = T::NT / BM_;
            float* part = reinterpret_cast<float*>(part_buf);
            part[tid] = rsum;
            __syncthreads();
            if (tid < BM_ && m0 + tid < M) {
                float t = part[tid];
#pragma unroll
                for (int q = 1; q < SPLIT; ++q) t += part[tid + q * BM_];
                p.bsum[static_cast<size_t>(e) * M + m0 + tid] = t;
            }
            __syncthreads();
        }
    }

    char* ep = reinterpret_cast<char*>(ep_buf);
    constexpr int SEG = 16 / ELEM;                 // elements per 16-byte segment
    constexpr int LANES_PER_ROW = WN / SEG;
    constexpr int ROWS_PER_PASS = 64 / LANES_PER_ROW;
    constexpr int PASSES = 32 / ROWS_PER_PASS;
    static_assert(64 % LANES_PER_ROW == 0 && WN % SEG == 0, "epilogue row split");

#pragma unroll
    for (int i = 0; i < FM; ++i) {
        if (i >= fm_live) break;  // the wave's remaining rows are past M
        // saved gelu'(H) of the block's rows, all loads in flight together
        uint2 aux[EPI == EPI_GELU_GRAD ? FN * 4 : 1];
        if constexpr (EPI == EPI_GELU_GRAD) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = n0 + wn * WN + j * 32 + 8 * q + 4 * (lane >> 5);
                    const int m = m0 + wm * WM + i * 32 + (lane & 31);
                    aux[j * 4 + q] = (n < N && m < M)
                                         ? *reinterpret_cast<const uint2*>(
                                               static_cast<const uint16_t*>(p.aux) +
                                               e * p.out_estride + static_cast<size_t>(m) * p.ldo + n)
                                         : make_uint2(0u, 0u);
                }
        }
        // Stage 1: register 4q + r of lane l holds C[m][n + r] with m = 32 i + l % 32,
        // n = 32 j + 8 q + 4 (l / 32) inside the wave tile.
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ml = lane & 31;  // row inside the staged rows
                const int nl = j * 32 + 8 * q + 4 * (lane >> 5);
                const f32x16& v = acc[i][j];
                float r[4] = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                if constexpr (F32_OUT) {
                    *reinterpret_cast<float4*>(reinterpret_cast<float*>(ep) + ml * EP_LD + nl) =
                        make_float4(r[0], r[1], r[2], r[3]);
                } else {
                    // (the bias of EPI_FWD1 / EPI_BIAS is already in acc)
                    if constexpr (EPI == EPI_GELU_GRAD) {
                        const uint2 gg = aux[j * 4 + q];
                        r[0] *= bf16_to_f32(gg.x & 0xFFFFu);
                        r[1] *= bf16_to_f32(gg.x >> 16);
                        r[2] *= bf16_to_f32(gg.y & 0xFFFFu);
                        r[3] *= bf16_to_f32(gg.y >> 16);
                    }
                    uint16_t* t0 = reinterpret_cast<uint16_t*>(ep) + ml * EP_LD + nl;
                    if constexpr (EPI == EPI_FWD1) {
                        float g[4], dg[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) gelu_pair(r[c], g[c], dg[c]);
                        *reinterpret_cast<uint2*>(t0 + EP_TILE / 2) =
                            make_uint2(pack_bf16x2(dg[0], dg[1]), pack_bf16x2(dg[2], dg[3]));
#pragma unroll
                        for (int c = 0; c < 4; ++c) r[c] = g[c];
                    }
                    *reinterpret_cast<uint2*>(t0) =
                        make_uint2(pack_bf16x2(r[0], r[1]), pack_bf16x2(r[2], r[3]));
                }
            }

        // Stage 2: staged rows out in 16-byte segments.
        const int cl = (lane % LANES_PER_ROW) * SEG;
        const int n = n0 + wn * WN + cl;
#pragma unroll
        for (int o = 0; o < OUTS; ++o) {
            char* dst_base = static_cast<char*>(o == 0 ? p.out : p.out2);
#pragma unroll
            for (int pass = 0; pass < PASSES; ++pass) {
                const int ml = pass * ROWS_PER_PASS + lane / LANES_PER_ROW;
                const int m = m0 + wm * WM + i * 32 + ml;
                const uint4 v =
                    *reinterpret_cast<const uint4*>(ep + o * EP_TILE + (ml * EP_LD + cl) * ELEM);
                if (m < M && n < N) {
                    v4i32* dst = reinterpret_cast<v4i32*>(
                        dst_base + (e * p.out_estride + static_cast<size_t>(m) * p.ldo + n) * ELEM);
                    // weight gradients are not read again by the layer: streaming
                    // stores keep them from displacing cached activations (the f32
                    // write-back cost a fifth of the weight-gradient GEMM, measured alone)
                    if constexpr (F32_OUT)
                        __builtin_nontemporal_store(__builtin_bit_cast(v4i32, v), dst);
                    else
                        *dst = __builtin_bit_cast(v4i32, v);
                }
            }
        }
    }
}

// Light tiles. A tile whose live rows fit one 32-row block (an expert with a
// handful of rows under a skewed load) streams a BN-column weight panel over
// the whole k range for a few products, so its time is that stream, and the
// stage ring keeps only NS - 1 stages of it in flight. Such a tile skips the
// ring: each wave streams its own share in 64-deep k groups, two groups in
// flight in registers, every load a coalesced 128-byte piece of a row; a
// group passes through a small LDS block of the wave's own to be read back
// as fragments. The waves of the block split the tile's columns (whole wave
// columns) and its k groups between them, and the waves of k slice 0 add the
// other slices' sums in slice order (a fixed order) before the usual
// epilogue of their one live row block.
constexpr int kLightGroups = 2;  // 64-deep k groups in flight per wave

// LDS-typed views of a tile's arrays (a pointer selected
// among the arrays at run time would otherwise become a flat pointer, whose
// accesses wait on the vector-memory counter too)
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) v4i32 lds_v4;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) float lds_f32;

// A phased tile's LDS arrays, and their eight 16 KB pieces (a select over values:
// a closure or array of the arrays' addresses would sit in scratch memory)
struct LdsArrays {
    uint16_t *b0, *b1, *b2, *b3, *b4, *b5, *b6;
};
__device__ __forceinline__ lds_u16* pick_lds(int i, const LdsArrays& a) {
    uint16_t* b = a.b0;
    if (i == 1) b = a.b0 + 8192;
    if (i == 2) b = a.b1;
    if (i == 3) b = a.b1 + 8192;
    if (i == 4) b = a.b6;
    if (i == 5) b = a.b6 + 8192;
    if (i == 6) b = a.b2;
    if (i == 7) b = a.b4;
    return (lds_u16*)(b);
}

template <class T, bool A_KMAJOR, bool B_KMAJOR, int EPI>
constexpr bool light_ok() {
    return A_KMAJOR && EPI != EPI_F32 && T::WN == 64;
}

// A light expert's tiles split into this many column parts (whole wave
// columns each, so the parts divide T's wave columns), of at most `slots`, the
// expert's m-tile slots of the grid: one HBM stream per CU runs at a fraction
// of a CU's share of the chip's bandwidth, so a light tile's weight panel is
// spread over CUs.
template <class T>
__device__ __forceinline__ int light_parts(int slots) {
    if (T::WGN % 4 == 0 && slots >= 4) return 4;
    if (T::WGN % 3 == 0 && slots >= 3) return 3;
    if (T::WGN % 2 == 0 && slots >= 2) return 2;
    return 1;
}

template <class T>
struct LightOf {
    using type = T;
};
template <int PB>
struct LightOf<PhaseTile<PB>> {
    using type = LightShape<PB>;
};

template <class T, class CFG, bool B_KMAJOR, int EPI, int GS>
__device__ __forceinline__ void light_tile(const GemmArgs& p, __amdgpu_buffer_rsrc_t ra_rs,
                                           __amdgpu_buffer_rsrc_t rb_rs, int e, int M, int N,
                                           int K, int m0, int n0, int part, int nparts,
                                           const LdsArrays& arrays) {
    constexpr int FM = T::FM, FN = T::FN, WN = T::WN, WGN = T::WGN;
    constexpr int U = kLightGroups;
    constexpr int LD = 64 + 8;          // LDS row: 64 elements + 16 bytes (rows on other banks)
    constexpr int A_EL = 32 * LD;       // A block: 32 rows x 64 k
    constexpr int B_EL = 64 * LD;       // B block: 64 n x 64 k (k-major) or 64 k x 64 n
    constexpr int W_EL = A_EL + B_EL;   // one wave's LDS block
    constexpr int PB = FN * 16 * 64;    // floats of one wave's partial sums
    static_assert(WN == 64 && FN == 2, "light tiles: 64-column wave tiles");
    static_assert(W_EL * 2 <= CFG::BUF_BYTES && PB * 4 <= CFG::BUF_BYTES,
                  "a wave's LDS block and its partial sums fit its buffer");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the part's columns are `cols` wave columns; wave w takes column c and k
    // slice sl of ks (slice 0 holds the sums)
    const int cols = WGN / nparts, ks = T::NW / cols;
    const int c = wave % cols, sl = wave / cols;
    const int nb = n0 + (part * cols + c) * WN;  // the wave's first column
    // the epilogue places wave w's columns at n0 + (w mod WGN) WN
    const int wn = wave % WGN, n0w = nb - wn * WN;
    // slice sl takes the 64-deep k groups [g0, g1); loads past klim read zeros
    const int ng = (K + 63) / 64;
    // (three columns leave waves past the last slice: no groups)
    const int g0 = ng * min(sl, ks) / ks, g1 = ng * min(sl + 1, ks) / ks;
    const int klim = min(K, g1 * 64);
    // load i of a group: row (k-major) or k row (mn-major) 8 i + lane / 8,
    // elements 8 (lane % 8) .. + 7 of its 64
    const int lr = lane >> 3, lc = 8 * (lane & 7);
    int arow[4];  // element offsets of the lane's A rows, -1 past M
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int mr = m0 + 8 * i + lr;
        if constexpr (GS == 1) arow[i] = mr < M ? p.tok[e * p.tok_estride + mr] * p.a.ld : -1;
        else arow[i] = mr < M ? mr * p.a.ld : -1;
    }

    uint4 ra[U][4], rb[U][8];
    auto load = [&](int u, int g) {
        const int k = g * 64 + lc;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            ra[u][i] = buf_load16(ra_rs, arow[i] >= 0 && k < klim
                                             ? static_cast<uint32_t>(arow[i] + k) * 2u
                                             : kOutOfRange);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (B_KMAJOR)
                rb[u][i] = buf_load16(rb_rs, vec_off<true>(p.b.ld, nb + 8 * i + lr, N, k, klim));
            else
                rb[u][i] = buf_load16(rb_rs, vec_off<false>(p.b.ld, nb + lc, N, g * 64 + 8 * i + lr,
                                                            klim));
        }
    };

    BiasRegs<T, EPI> bias;
    bias.load(p, e, N, n0w, wn, lane);
    f32x16 lacc[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float b4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (BiasRegs<T, EPI>::USED) {
                if (sl == 0) {
                    const uint2 bb = bias.v[j * 4 + q];
                    b4[0] = bf16_to_f32(bb.x & 0xFFFFu);
                    b4[1] = bf16_to_f32(bb.x >> 16);
                    b4[2] = bf16_to_f32(bb.y & 0xFFFFu);
                    b4[3] = bf16_to_f32(bb.y >> 16);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) lacc[j][4 * q + r] = b4[r];
        }

    // wave w's LDS block: buffer w
    lds_u16* const as = pick_lds(wave, arrays);
    lds_u16* const bs = as + A_EL;
    // (group by group, as the loop refills them: each group then waits for its
    // own loads only, also on the loop's first trip)
#pragma unroll
    for (int u = 0; u < U; ++u) {
        load(u, g0 + u);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int g = g0; g < g1; g += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // the group into the wave's LDS block (one wave's LDS accesses run
            // in order: the previous group's fragment reads are done first)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<lds_v4*>(as + (8 * i + lr) * LD + lc) =
                    __builtin_bit_cast(v4i32, ra[u][i]);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                *reinterpret_cast<lds_v4*>(bs + (8 * i + lr) * LD + lc) =
                    __builtin_bit_cast(v4i32, rb[u][i]);
            __builtin_amdgcn_sched_barrier(0);
            // its registers refill with group g + u + U (past g1: out of range,
            // no traffic), so U groups stay in flight
            load(u, g + u + U);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int kk = 16 * s + 8 * (lane >> 5);
                const bf16x8 a = *reinterpret_cast<const lds_bf16x8*>(as + (lane & 31) * LD + kk);
                bf16x8 b[FN];
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    if constexpr (B_KMAJOR) {
                        b[j] = *reinterpret_cast<const lds_bf16x8*>(bs + (32 * j + (lane & 31)) * LD +
                                                                    kk);
                    } else {
                        // transposing reads of the [k][n] block: lane gets column
                        // 32 j + lane % 32, k rows 16 s + 8 (lane / 32) + 0..7
                        const int gq = lane >> 4, jj = lane & 15;
                        const int kr = 16 * s + 8 * (gq >> 1) + (jj >> 2);
                        const int n = 32 * j + 16 * (gq & 1) + 4 * (jj & 3);
                        typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
                        const s16x4 lo =
                            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(bs + kr * LD + n));
                        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (lds_s16x4)(bs + (kr + 4) * LD + n));
                        b[j] = __builtin_bit_cast(
                            bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                    }
                }
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    lacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a, lacc[j], 0, 0, 0);
            }
        }
    }

    // slices 1.. park their sums (slice sl, column c: buffer (sl - 1) cols + c);
    // every wave is past its LDS block first
    auto slot = [&](int s) { return reinterpret_cast<lds_f32*>(pick_lds(s, arrays)); };
    __syncthreads();
    if (sl > 0) {
        lds_f32* const dst = slot((sl - 1) * cols + c);
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) dst[(j * 16 + r) * 64 + lane] = lacc[j][r];
    }
    __syncthreads();
    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    if (sl == 0) {
        for (int s = 1; s < ks; ++s) {
            const lds_f32* const src = slot((s - 1) * cols + c);
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) lacc[j][r] += src[(j * 16 + r) * 64 + lane];
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[0][j] = lacc[j];
    }
    __syncthreads();  // the sums are read before the epilogue stages outputs over them
    uint16_t* const ep = (uint16_t*)(pick_lds(wave, arrays));  // (an LDS pointer, seen as such)
    gemm_epilogue<T, CFG, EPI>(p, acc, arrays.b0, ep, 0.0f, false, e, M, N, m0, n0w, sl == 0 ? 1 : 0);
}

// Epilogue of a phased tile with bf16 outputs: each wave turns its accumulators
// into outputs strip by strip (64 rows x 32 columns of panel b), through 4 KB of
// LDS of its own, 16-byte chunks XOR-swizzled by row, to be stored as 64-byte row
// segments. A wave's LDS accesses run in order, so no pass needs a barrier, and
// the operand stages are not touched. The saved gelu'(H) arrives in the same row
// segments, all strips requested before the first is used.
template <class T, int EPI>
__device__ __forceinline__ void phase_epilogue(const GemmArgs& p, f32x16 (&acc)[T::FM][T::PB],
                                               uint16_t* stg, int e, int M, int N, int m0, int n0,
                                               int fm_live) {
    static_assert(EPI != EPI_F32, "bf16 outputs");
    constexpr int PB = T::PB, FM = T::FM;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    const int mr = m0 + 64 * wm, nc = n0 + 32 * wn;  // the wave's first row and column
    if (fm_live == 0) return;
    typedef int v2i32 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) v2i32 lds_v2;
    lds_u16* const s = (lds_u16*)(stg) + wave * 2048;
    const size_t ebase = static_cast<size_t>(e) * p.out_estride;
    // lane's row segment u of a strip: row 16 u + lane / 4, chunk lane % 4
    const int sr = lane >> 2, sc = lane & 3;
    auto slot = [&](int r, int c) { return s + r * 32 + ((c ^ ((r >> 2) & 3)) << 3); };
    v4i32 aux[EPI == EPI_GELU_GRAD ? PB : 1][4];
    if constexpr (EPI == EPI_GELU_GRAD) {
#pragma unroll
        for (int b = 0; b < PB; ++b)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int m = mr + 16 * u + sr, n = nc + 64 * b + 8 * sc;
                aux[b][u] = (m < M && n < N)
                                ? *reinterpret_cast<const v4i32*>(
                                      static_cast<const uint16_t*>(p.aux) + ebase +
                                      static_cast<size_t>(m) * p.ldo + n)
                                : v4i32{0, 0, 0, 0};
            }
    }
    // the staged strip to `dst` as row segments
    auto rows_out = [&](int b, void* dst) {
        const int n = nc + 64 * b + 8 * sc;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int m = mr + 16 * u + sr;
            const v4i32 v = *reinterpret_cast<lds_v4*>(slot(16 * u + sr, sc));
            if (m < M && n < N)
                *reinterpret_cast<v4i32*>(static_cast<uint16_t*>(dst) + ebase +
                                          static_cast<size_t>(m) * p.ldo + n) = v;
        }
    };
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        uint2 dg[EPI == EPI_FWD1 ? FM : 1][4];
        if constexpr (EPI == EPI_GELU_GRAD) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                *reinterpret_cast<lds_v4*>(slot(16 * u + sr, sc)) = aux[b][u];
        }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float r[4] = {acc[i][b][4 * q], acc[i][b][4 * q + 1], acc[i][b][4 * q + 2],
                              acc[i][b][4 * q + 3]};
                lds_u16* const at = slot(32 * i + (lane & 31), q) + 4 * (lane >> 5);
                if constexpr (EPI == EPI_GELU_GRAD) {
                    const v2i32 gg = *reinterpret_cast<lds_v2*>(at);
                    r[0] *= bf16_to_f32(gg[0] & 0xFFFFu);
                    r[1] *= __uint_as_float(gg[0] & 0xFFFF0000u);
                    r[2] *= bf16_to_f32(gg[1] & 0xFFFFu);
                    r[3] *= __uint_as_float(gg[1] & 0xFFFF0000u);
                }
                if constexpr (EPI == EPI_FWD1) {
                    float g[4], d[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) gelu_pair(r[c], g[c], d[c]);
                    dg[i][q] = make_uint2(pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3]));
#pragma unroll
                    for (int c = 0; c < 4; ++c) r[c] = g[c];
                }
                *reinterpret_cast<lds_v2*>(at) =
                    v2i32{static_cast<int>(pack_bf16x2(r[0], r[1])),
                          static_cast<int>(pack_bf16x2(r[2], r[3]))};
            }
        rows_out(b, p.out);
        if constexpr (EPI == EPI_FWD1) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<lds_v2*>(slot(32 * i + (lane & 31), q) +
                                               4 * (lane >> 5)) =
                        v2i32{static_cast<int>(dg[i][q].x), static_cast<int>(dg[i][q].y)};
            rows_out(b, p.out2);
        }
    }
}

// Epilogue of a phased weight-gradient tile. Where rows are whole 128-byte lines,
// strip by strip as above: a 32-row block's 32 columns of a panel, one line a row,
// without a barrier. Elsewhere such strips write every line in two parts, so whole
// rows of the tile go out instead, a row an instruction: in pass i every wave puts
// its 32-row block i of all panels into the tile's arrays, whose operands are done
// with (16 rows to a 16 KB piece), and wave w stores the 16 rows of piece w.
// Measured, expert MLP backward with strips / whole rows: 8 rows an expert, E = 64,
// d = 1000, f = 2000 454 / 335 us (365 with the former 256-byte segments of a wave);
// 30 rows, E = 64, d = 520, f = 2088 329 / 244 (255); 64 rows, E = 32, d = 1024,
// f = 4096 (whole lines) 337 / 341 (385); 768 x 3072 207 / 213 (229).
template <class T>
__device__ __forceinline__ void phase_epilogue_f32(const GemmArgs& p,
                                                   f32x16 (&acc)[T::FM][T::PB],
                                                   float (&rsum)[T::FM], bool row_sum,
                                                   const LdsArrays& arrays, int e, int M, int N,
                                                   int m0, int n0, int fm_live) {
    constexpr int PB = T::PB, FM = T::FM, ROW = 128 * PB;  // a staged row, in 16-bit words
    // (opaque, so that the quota schedule's loop over tiles does not carry the
    // addresses below through its products: 30 spilled registers, ViT-L/16 step
    // under quotas 1352 us against 1325)
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int wave = wave_id();
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    const int mr = m0 + 64 * wm;
    if (row_sum) {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const float t = rsum[i] + __shfl_xor(rsum[i], 32, 64);
            const int m = mr + 32 * i + lane;
            if (lane < 32 && m < M) p.bsum[static_cast<size_t>(e) * M + m] = t;
        }
    }
    float* const out = static_cast<float*>(p.out) + static_cast<size_t>(e) * p.out_estride;
    // chunk q (4 columns) of the lane's row in block i, panel b
    auto chunk = [&](int i, int b, int q) {
        return __builtin_bit_cast(v4i32, make_float4(acc[i][b][4 * q], acc[i][b][4 * q + 1],
                                                     acc[i][b][4 * q + 2], acc[i][b][4 * q + 3]));
    };
    // weight gradients are not read again by the layer: streaming stores keep
    // them from displacing cached activations
    auto store = [&](v4i32 v, int m, int n) {
        __builtin_nontemporal_store(
            v, reinterpret_cast<v4i32*>(out + static_cast<size_t>(m) * p.ldo + n));
    };
    if (p.ldo % 32 == 0) {
        if (fm_live == 0) return;
        lds_u16* const s = (lds_u16*)(arrays.b6) + wave * 2048;
        const int nc = n0 + 32 * wn;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            if (i >= fm_live) break;
#pragma unroll
            for (int b = 0; b < PB; ++b) {
                // row r of the staged block: 8 chunks of 16 bytes
                const int r = lane & 31;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = 2 * q + (lane >> 5);
                    *reinterpret_cast<lds_v4*>(s + r * 64 + ((c ^ (r & 7)) << 3)) = chunk(i, b, q);
                }
                const int n = nc + 64 * b + 4 * (lane & 7);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int rr = 8 * u + (lane >> 3), m = mr + 32 * i + rr;
                    const v4i32 v = *reinterpret_cast<lds_v4*>(
                        s + rr * 64 + (((lane & 7) ^ (rr & 7)) << 3));
                    if (m < M && n < N) store(v, m, n);
                }
            }
        }
        return;
    }
    lds_u16* const lo = pick_lds(2 * wm, arrays);
    lds_u16* const hi = pick_lds(2 * wm + 1, arrays);
    lds_u16* const mine = pick_lds(wave, arrays);
    const int r = lane & 15, n = n0 + 4 * lane;
    lds_u16* const put = ((lane & 16) ? hi : lo) + r * ROW;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        lds_barrier();  // the operands, or the previous pass's rows, are read
        if (i < fm_live) {
#pragma unroll
            for (int b = 0; b < PB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = 16 * b + 8 * wn + 2 * q + (lane >> 5);
                    *reinterpret_cast<lds_v4*>(put + ((c ^ r) << 3)) = chunk(i, b, q);
                }
        }
        lds_barrier();
        const int m1 = mr + 32 * i + 16 * wn;  // the wave's first row
        if (lane < 16 * PB && n < N) {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const v4i32 v = *reinterpret_cast<lds_v4*>(mine + u * ROW + ((lane ^ u) << 3));
                if (m1 + u < M) store(v, m1 + u, n);
            }
        }
    }
}

// One tile of a PhaseTile<PB>: wave w = (wm, wn) accumulates rows 64 wm .. + 63
// and, of every 64-column panel b, columns 32 wn .. + 31 (acc[i][b]: 32-row
// block i). A stage is 64 deep; its phase b multiplies the wave's A fragments
// (read once per stage) by panel b and meanwhile reads the next panel's
// fragments, in the last phase also the next stage's A fragments, each right
// after the last product that uses the old one.
//
// Every phase opens with a barrier, and a panel's LDS slot is refilled one
// phase after its fragments were used, so the loads of a stage go out a few
// at a time and early: with PB = 4, six phases (1.5 stages) before they
// are read, where a ring of two whole stages issued all eight of a wave's
// loads in one burst behind the barrier, ahead of the products, and needed
// them back within the stage. 4 x 2 waves and 64-column panels keep every
// row segment a whole 128-byte line in either layout (a ring of 32-deep
// stages fetches half lines and measured 10-20% slower). Measured against
// that ring, whose tiles were the same size: down-projection 306 -> 260 us,
// gelu'-product 396 -> 347 at 49 000 rows over 32 experts, d = 768, f = 3072
// (256 x 256); down-projection 140 -> 109, dxe beside the weight gradients
// 345 -> 291 on the 17-task batch (256 x 192). Matrix products alone (no
// loads, no LDS reads) take 156 of the 260, the rate the card holds on random
// data; waiting for all but half of the loads in flight costs 6%, so neither
// depth nor latency binds. Per phase a wave issues
//   phase 0: panel PB - 1 of stage kt + 1     phase 1: panel 0, A of stage kt + 2
//   phase b: panel b - 1 of stage kt + 2
// and waits before phase b for what phase b reads, counting what was issued
// after it. Every fragment read in a phase is used by the next phase's products
// (the last phase's A fragments by all of them in the next stage's phase 0), which
// the scheduling barriers keep ahead of the barrier that opens the phase after
// that: there alone may their LDS be refilled, without a wait for LDS reads.
// Only the last stage's read of a stage past K goes unused; nothing is requested
// after it. (A wave without live rows reads no fragments and only requests.)
template <int PB>
struct PhaseWaits {
    static constexpr int issued(int b) { return b == 1 ? 5 : 1; }  // wave instructions, phase b
    static constexpr int stage() { return PB + 4; }
    static constexpr int upto(int b) {  // of phases 0 .. b - 1
        int n = 0;
        for (int q = 0; q < b; ++q) n += issued(q);
        return n;
    }
    // Instructions that may be in flight when phase b opens. Phase b < PB - 1
    // reads panel b + 1 of its stage: issued in phase b + 2 of two stages
    // before (first of that phase's instructions), or, panel PB - 1, in phase 0
    // of the stage before. The last phase reads panel 0 and A of the next
    // stage, issued in phase 1 of the stage before.
    static constexpr int flight(int b) {
        if (b == PB - 1) return stage() - upto(2) + upto(b);
        if (b == PB - 2) return stage() - upto(1) + upto(b);
        return (stage() - upto(b + 2) - 1) + stage() + upto(b);
    }
};

template <class T, bool A_KMAJOR, bool B_KMAJOR, int EPI, int GS>
__device__ __forceinline__ void phase_tile(const GemmArgs& p, __amdgpu_buffer_rsrc_t ra_rs,
                                           __amdgpu_buffer_rsrc_t rb_rs, int e, int M, int N,
                                           int K, int m0, int n0, int tn, uint16_t* a0,
                                           uint16_t* a1, uint16_t* bl0, uint16_t* bh0,
                                           uint16_t* bl1, uint16_t* bh1, uint16_t* stg) {
    constexpr int PB = T::PB, KB = T::KB, FM = T::FM, P_EL = T::P_EL;
    using DA = DmaStage<T::BM, A_KMAJOR, KB, T::NT>;  // four wave instructions a stage
    using DB = DmaStage<64, B_KMAJOR, KB, T::NT>;     // one a panel
    static_assert(DA::PER == 4 && DB::PER == 1, "stage split");
    using W = PhaseWaits<PB>;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    // 32-row blocks of the wave's rows that lie inside M
    const int fm_live = min(FM, max(0, (M - m0 - wm * T::WM + 31) / 32));

    int arow[GS == 1 ? DA::PER : 1];
    uint32_t aoff[DA::PER], boff[PB];
    uint32_t* const tok_s = reinterpret_cast<uint32_t*>(stg);  // k-row gather's row table
    uint32_t bk = 0;
    if constexpr (GS == 1) {
#pragma unroll
        for (int q = 0; q < DA::PER; ++q) {
            const int r = DA::lane_row(q);
            arow[q] = m0 + r < M ? p.tok[e * p.tok_estride + m0 + r] * p.a.ld : -1;
        }
        DA::lane_offs_rows(arow, aoff);
    } else {
        DA::lane_offs(p.a.ld, m0, M, aoff);
    }
    if constexpr (GS == 2) {
        // the expert's k rows as byte offsets of their rows of x, and the
        // sentinel past K up to the last stage that is requested
        const int kfill = ((K + 2 * KB - 1) / (2 * KB) + 1) * 2 * KB;
        for (int i = tid; i < kfill; i += T::NT)
            tok_s[i] = i < K ? static_cast<uint32_t>(p.tok[e * p.tok_estride + i]) *
                                   (2u * static_cast<uint32_t>(p.b.ld))
                             : kGatherSentinel;
        __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        uint32_t o[1];
        if constexpr (GS == 2) DB::krow_cols(n0 + 64 * b, N, o);
        else DB::lane_offs(p.b.ld, n0 + 64 * b, N, o);
        boff[b] = o[0];
    }
    const uint32_t a_step = (A_KMAJOR ? KB : KB * p.a.ld) * 2;
    const uint32_t b_step = (B_KMAJOR ? KB : KB * p.b.ld) * 2;
    const int nk = (K + KB - 1) / KB;
    const int n_inside = K / KB;  // stages that lie inside K

    // requests of stage kt (inside K, or any: zeros past K)
    auto issue_a = [&](int kt, uint16_t* dst, auto inside) {
        if constexpr (decltype(inside)::value) DA::issue_inside(ra_rs, aoff, kt * a_step, dst);
        else if constexpr (GS == 1) DA::issue_rows(ra_rs, arow, kt * KB, K, dst);
        else DA::issue(ra_rs, p.a.ld, m0, M, kt * KB, K, dst);
    };
    // panel b of stage buffer S
    auto panel = [&](auto parity, int b) {
        constexpr int S = decltype(parity)::value;
        return b < 2 ? (S ? bl1 : bl0) + b * P_EL : (S ? bh1 : bh0) + (b - 2) * P_EL;
    };
    auto issue_b = [&](int kt, int b, auto parity, auto inside) {
        uint32_t o[1] = {boff[b]};
        uint16_t* const dst = panel(parity, b);
        if constexpr (GS == 2) {
            // panels of a stage are requested in order: its rows with panel 0
            if (b == 0) bk = tok_s[kt * KB + DB::lane_row(0)];
            const uint32_t ro[1] = {bk};
            DB::issue_krows(rb_rs, ro, o, dst);
        } else if constexpr (decltype(inside)::value) {
            DB::issue_inside(rb_rs, o, kt * b_step, dst);
        } else {
            DB::issue(rb_rs, p.b.ld, n0 + 64 * b, N, kt * KB, K, dst);
        }
    };
    using YES = std::true_type;
    using NO = std::false_type;

    // The bias of the wave's columns 64 b + 32 wn + 8 q + 4 (lane / 32) + 0..3
    // starts the accumulators.
    constexpr bool BIAS = EPI == EPI_FWD1 || EPI == EPI_BIAS;
    uint2 bias[BIAS ? PB * 4 : 1];
    if constexpr (BIAS) {
#pragma unroll
        for (int b = 0; b < PB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + 64 * b + 32 * wn + 8 * q + 4 * (lane >> 5);
                bias[b * 4 + q] = n < N ? *reinterpret_cast<const uint2*>(
                                              static_cast<const uint16_t*>(p.bias) +
                                              e * p.bias_estride + n)
                                        : make_uint2(0u, 0u);
            }
    }

    // the loop's first two stages, in the order the phases would have issued them
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    issue_b(0, 0, P0{}, NO{});
    issue_a(0, a0, NO{});
#pragma unroll
    for (int b = 1; b < PB; ++b) issue_b(0, b, P0{}, NO{});
    issue_b(1, 0, P1{}, NO{});
    issue_a(1, a1, NO{});
#pragma unroll
    for (int b = 1; b < PB - 1; ++b) issue_b(1, b, P1{}, NO{});

    f32x16 acc[FM][PB];
#pragma unroll
    for (int b = 0; b < PB; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float b4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (BIAS) {
                const uint2 bb = bias[b * 4 + q];
                b4[0] = bf16_to_f32(bb.x & 0xFFFFu);
                b4[1] = bf16_to_f32(bb.x >> 16);
                b4[2] = bf16_to_f32(bb.y & 0xFFFFu);
                b4[3] = bf16_to_f32(bb.y >> 16);
            }
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][b][4 * q + r] = b4[r];
        }

    // bias gradients: the first n-tile's waves of column half 0 also sum
    // their A rows (dot products with ones, from the fragments)
    const bool row_sum = EPI == EPI_F32 && p.bsum != nullptr && tn == 0 && wn == 0;
    float rsum[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) rsum[i] = 0.0f;

    // A and panel 0 of stage 0 have landed
    __builtin_amdgcn_s_waitcnt(VmWait<W::flight(PB - 1) + W::issued(PB - 1)>::imm | (15 << 8));
    ring_barrier();

    auto ring = [&](auto live_blocks) {
        constexpr int FL = decltype(live_blocks)::value;
        bf16x8 fa[FM][4], fb[2][4];
        auto read_a = [&](const uint16_t* as, int ks) {
#pragma unroll
            for (int i = 0; i < FL; ++i)
                fa[i][ks] = read_frag<T::BM, A_KMAJOR, KB>(as, wm * FM + i, ks, lane);
        };
        if constexpr (FL > 0) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                read_a(a0, ks);
                fb[0][ks] = read_frag<64, B_KMAJOR, KB>(bl0, wn, ks, lane);
            }
        }
        // stage kt: A in ac, the next stage's in an; S = kt mod 2
        auto stage = [&](int kt, uint16_t* ac, uint16_t* an, auto parity, auto inside) {
            constexpr int S = decltype(parity)::value;
            using NX = std::integral_constant<int, 1 - S>;
            auto phase = [&](auto which) {
                constexpr int b = decltype(which)::value;
                constexpr int cur = (S * PB + b) & 1;
                __builtin_amdgcn_s_waitcnt(VmWait<W::flight(b)>::imm | (15 << 8));
                ring_barrier();
                const uint16_t* bs = b < PB - 1 ? panel(parity, b + 1) : panel(NX{}, 0);
                auto products = [&](int ks) {
#pragma unroll
                    for (int i = 0; i < FL; ++i)
                        acc[i][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            fb[cur][ks], fa[i][ks], acc[i][b], 0, 0, 0);
                };
                auto next_b = [&](int ks) {
                    if constexpr (FL > 0)
                        fb[cur ^ 1][ks] =
                            read_frag<64, B_KMAJOR, KB>(bs, wn, ks, lane);
                };
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    products(ks);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (b == PB - 1) {
                        if constexpr (EPI == EPI_F32) {
                            if (row_sum) {
#pragma unroll
                                for (int i = 0; i < FL; ++i) {
                                    const bf16x8 v = fa[i][ks];
#pragma unroll
                                    for (int c = 0; c < 8; ++c)
                                        rsum[i] += static_cast<float>(v[c]);
                                }
                            }
                        }
                        read_a(an, ks);
                        next_b(ks);
                    } else if (ks < 2) {
                        next_b(2 * ks);
                        next_b(2 * ks + 1);
                    }
                    // this phase's requests
                    if (ks == 0) {
                        if constexpr (b == 0) issue_b(kt + 1, PB - 1, NX{}, inside);
                        else issue_b(kt + 2, b - 1, parity, inside);
                    }
                    if constexpr (b == 1)
                        if (ks == 1) issue_a(kt + 2, ac, inside);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            phase(std::integral_constant<int, 0>{});
            phase(std::integral_constant<int, 1>{});
            if constexpr (PB > 2) phase(std::integral_constant<int, 2>{});
            if constexpr (PB > 3) phase(std::integral_constant<int, 3>{});
        };
        int kt = 0;
        for (; kt + 3 < n_inside; kt += 2) {
            stage(kt, a0, a1, P0{}, YES{});
            stage(kt + 1, a1, a0, P1{}, YES{});
        }
        // (an odd last stage runs alone: with a stage of zeros after it an expert of
        // at most 64 rows paid for two stages of weight gradients, backward at 64
        // rows, E = 64, d = 1008, f = 2016 358 us against 339)
        for (; kt < nk; kt += 2) {
            stage(kt, a0, a1, P0{}, NO{});
            if (kt + 1 < nk) stage(kt + 1, a1, a0, P1{}, NO{});
        }
    };
    if (fm_live > 1) ring(std::integral_constant<int, 2>{});
    else if (fm_live > 0) ring(std::integral_constant<int, 1>{});
    else ring(std::integral_constant<int, 0>{});
    // the requests past K have landed (here, so that no wait stands behind the stores)
    __builtin_amdgcn_s_waitcnt(VmWait<0>::imm | (15 << 8));
    if constexpr (EPI == EPI_F32)
        phase_epilogue_f32<T>(p, acc, rsum, row_sum, LdsArrays{a0, a1, bl0, bh0, bl1, bh1, stg}, e, M,
                              N, m0, n0, fm_live);
    else
        phase_epilogue<T, EPI>(p, acc, stg, e, M, N, m0, n0, fm_live);
}

// One SmallTile of a weight gradient: wave w = (wm, wn) accumulates 64 x 64 as 32 x 32
// blocks. Pipeline over 32-deep k-stages, one barrier per stage, four stage buffers
// (separate LDS arrays, so every access names its buffer statically):
//   issue the loads of stage kt + 3 (into the buffer that stage kt - 1 used)
//   read fragments of step 1                      | MFMAs of step 0
//   wait until stage kt + 1 has landed; barrier
//   read step-0 fragments of stage kt + 1         | MFMAs of step 1
// so LDS latency always hides behind a run of MFMAs on held fragments, and
// HBM latency behind three stages of MFMAs. The stage count is rounded up to
// a multiple of four so the ring unrolls with static buffers; the padding
// stages load zeros (out of range) and skip their MFMAs.
// GS = 2: operand B's k rows are gathered.
template <int GS>
__device__ __forceinline__ void ring_tile(const GemmArgs& p, __amdgpu_buffer_rsrc_t ra_rs,
                                          __amdgpu_buffer_rsrc_t rb_rs, int e, int M, int N, int K,
                                          int m0, int n0, int tn, uint16_t* buf0, uint16_t* buf1,
                                          uint16_t* buf2, uint16_t* buf3, uint32_t* tok_s) {
    using T = SmallTile;
    using CFG = GemmCfg<T, EPI_F32>;
    constexpr int KB = T::KB, NS = T::NS, NT = T::NT, FM = T::FM, FN = T::FN;
    constexpr int KSTEPS = T::KSTEPS, AE = T::BM * KB;
    static_assert(NS == 4 && KSTEPS == 2, "the ring below");
    using DA = DmaStage<T::BM, false, KB, NT>;
    using DB = DmaStage<T::BN, false, KB, NT>;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = wave_id();
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    // 32-row blocks of this wave's rows that lie inside M
    const int fm_live = __builtin_amdgcn_readfirstlane(
        min(FM, max(0, (M - m0 - wm * T::WM + 31) / 32)));
    // Gathered k rows (new ones every stage): the expert's token list in LDS, each
    // lane's offsets for the next stage read one stage ahead.
    uint32_t bk[GS == 2 ? DB::PER : 1], bcol[GS == 2 ? DB::PER : 1];
    if constexpr (GS == 2) {
        // the expert's k rows as byte offsets of their rows of x, and the
        // sentinel past K up to the last row the ring prefetches (so the
        // stage loop tests no bound)
        const int kfill = ((K + NS * KB - 1) / (NS * KB) + 1) * NS * KB;
        for (int i = tid; i < kfill; i += NT)
            tok_s[i] = i < K ? static_cast<uint32_t>(p.tok[e * p.tok_estride + i]) *
                                   (2u * static_cast<uint32_t>(p.b.ld))
                             : kGatherSentinel;
        __syncthreads();
        DB::krow_cols(n0, N, bcol);
#pragma unroll
        for (int q = 0; q < DB::PER; ++q) bk[q] = tok_s[DB::lane_row(q)];
    }
    // the first n-tile also sums its A rows (bias gradient): thread t adds row
    // t % BM over k slice t / BM of each stage
    const bool row_sum = p.bsum != nullptr && tn == 0;
    constexpr int RS_K = KB / (NT / T::BM);
    float rsum = 0.0f;

    // DMA wave instructions per stage; stage kt + 1 has landed once at most
    // NS - 2 later stages are still in flight
    constexpr int WAIT_IMM = VmWait<(NS - 2) * (DA::PER + DB::PER)>::imm;
    const int nk = (K + KB - 1) / KB;
    const int nk_ring = (nk + NS - 1) / NS * NS;
    // stages [0, n_inside) lie inside K: their loads differ in a scalar only
    // (the k-row gather has new rows every stage)
    const int n_inside = K / KB;
    uint32_t aoff[DA::PER], boff[DB::PER];
    DA::lane_offs(p.a.ld, m0, M, aoff);
    if constexpr (GS != 2) DB::lane_offs(p.b.ld, n0, N, boff);
    const uint32_t a_step = KB * p.a.ld * 2, b_step = KB * p.b.ld * 2;
    auto issue = [&](int kt, uint16_t* dst) {
        const bool inside = kt < n_inside;
        if (inside) DA::issue_inside(ra_rs, aoff, kt * a_step, dst);
        else DA::issue(ra_rs, p.a.ld, m0, M, kt * KB, K, dst);
        if constexpr (GS == 2) {
            DB::issue_krows(rb_rs, bk, bcol, dst + AE);
            // stages are issued in order: the next one's k rows
#pragma unroll
            for (int q = 0; q < DB::PER; ++q) bk[q] = tok_s[(kt + 1) * KB + DB::lane_row(q)];
        } else {
            if (inside) DB::issue_inside(rb_rs, boff, kt * b_step, dst + AE);
            else DB::issue(rb_rs, p.b.ld, n0, N, kt * KB, K, dst + AE);
        }
    };
    issue(0, buf0);
    issue(1, buf1);
    issue(2, buf2);
    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    __builtin_amdgcn_s_waitcnt(WAIT_IMM);
    ring_barrier();

    // The stage loop of a wave with FL row blocks to compute: straight-line,
    // instantiated for both, one and none of the blocks, since a test per row block
    // inside the loop would make every block a branch, at which the compiler waits
    // for the fragments in flight; blocks past the rows of the output are computed
    // on whatever the stage holds and never stored. Every instantiation meets the
    // same barriers.
    Frags<T> f0, f1;
    auto ring = [&](auto live_blocks) {
        constexpr int FL = decltype(live_blocks)::value;
        f0.template read<FL>(buf0, buf0 + AE, wm, wn, 0, lane);
        // stage kt computes from `cur`, refills `tgt` (the buffer of stage kt - 1)
        // and leaves the step-0 fragments of `nxt` in f0
        auto stage = [&](const int kt, uint16_t* cur, uint16_t* nxt, uint16_t* tgt) {
            issue(kt + NS - 1, tgt);
            const bool live = kt < nk;  // uniform: ring padding stages skip their MFMAs
            if (live) {
                if (row_sum) {
                    const int mn = tid % T::BM, k0 = (tid / T::BM) * RS_K;
#pragma unroll
                    for (int kk = 0; kk < RS_K; ++kk)
                        rsum += bf16_to_f32(cur[lds_off<T::BM, false, KB>(mn, k0 + kk)]);
                }
                f1.template read<FL>(cur, cur + AE, wm, wn, 1, lane);
                __builtin_amdgcn_sched_barrier(0);
                mfma_block<FL>(acc, f0);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_waitcnt(WAIT_IMM);
            ring_barrier();
            if (live) {
                f0.template read<FL>(nxt, nxt + AE, wm, wn, 0, lane);
                __builtin_amdgcn_sched_barrier(0);
                mfma_block<FL>(acc, f1);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // The ring unrolls four stages per trip with no conditional stage: a skipped
        // stage would merge a path with loads still in flight into the loop head.
        for (int kt = 0; kt < nk_ring; kt += NS) {
            stage(kt, buf0, buf1, buf3);
            stage(kt + 1, buf1, buf2, buf0);
            stage(kt + 2, buf2, buf3, buf1);
            stage(kt + 3, buf3, buf0, buf2);
        }
    };
    if (fm_live > 1) ring(std::integral_constant<int, 2>{});
    else if (fm_live > 0) ring(std::integral_constant<int, 1>{});
    else ring(std::integral_constant<int, 0>{});
    // every wave is done with the operand stages (LDS reads retired, DMA landed)
    __builtin_amdgcn_s_waitcnt(VmWait<0>::imm);
    ring_barrier();

    // wave w parks its outputs in stage buffer w (a select over the arrays
    // themselves keeps the accesses in the LDS address space)
    uint16_t* const ep = wave == 0 ? buf0 : wave == 1 ? buf1 : wave == 2 ? buf2 : buf3;
    gemm_epilogue<T, CFG, EPI_F32>(p, acc, buf0, ep, rsum, row_sum, e, M, N, m0, n0, fm_live);
}

// Elements of the kernel's LDS arrays.
template <class T, bool A_KMAJOR, bool B_KMAJOR, int EPI, int GATHER>
constexpr int gemm_lds(int i) {
    if constexpr (T::PHASED) {
        static_assert(GATHER != 2 || (kGatherRows + 4 * T::KB) * 2 <= T::S_EL,
                      "the gathered rows fit the epilogue's staging");
        const int n[7] = {T::A_EL,  T::A_EL,  T::BL_EL, T::BH_EL,
                          T::BL_EL, T::BH_EL, T::S_EL};
        return i < 7 ? n[i] : 1;
    } else {
        if (i < 7) return i < T::NS ? T::RING_BYTES / T::NS / 2 : 8;
        return GATHER == 2 ? kGatherRows + 2 * T::NS * T::KB : 1;
    }
}
template <class T, bool A_KMAJOR, bool B_KMAJOR, int EPI, int GATHER>
struct GemmLds {
    static constexpr int n(int i) { return gemm_lds<T, A_KMAJOR, B_KMAJOR, EPI, GATHER>(i); }
    static constexpr int B0 = n(0), B1 = n(1), B2 = n(2), B3 = n(3), B4 = n(4), B5 = n(5),
                         B6 = n(6), TOK = n(7);
};

// (the k-row gather's token table takes the LDS of a second 4-wave block)
template <class T, int GATHER>
constexpr int gemm_waves_per_eu() {
    return GATHER == 2 && T::NW == 4 ? 1 : T::WAVES_PER_EU;
}

// The bf16 GEMM kernel: one output tile of expert e per block; tiles are dealt to
// the 8 XCDs in chunks of neighbouring tiles (shared operand panels in each XCD's
// L2).
// SCHED = 0: one tile per block, the grid dealt over the (live) tile list;
// SCHED = 1: persistent blocks, each expert owning the number of blocks the
// fill-clamp-refill quota gives it, each block taking every units-th tile
// of its expert.
// GATHER = 1: operand A's rows are gathered token rows of x (the
// up-projection fused with the dispatch); GATHER = 2: operand B's k rows are
// (the input-weight gradient, problems with a token list).
template <class T, bool A_KMAJOR, bool B_KMAJOR, int EPI, int SCHED = 0, int GATHER = 0>
__global__ __launch_bounds__(T::NT)
__attribute__((amdgpu_waves_per_eu(gemm_waves_per_eu<T, GATHER>(),
                                   gemm_waves_per_eu<T, GATHER>())))
void gemm_bf16_kernel(GemmBatch batch) {
    constexpr int BM_ = T::BM, BN_ = T::BN;
    using LD = GemmLds<T, A_KMAJOR, B_KMAJOR, EPI, GATHER>;
    __shared__ __attribute__((aligned(1024))) uint16_t buf0[LD::B0];
    __shared__ __attribute__((aligned(1024))) uint16_t buf1[LD::B1];
    __shared__ __attribute__((aligned(1024))) uint16_t buf2[LD::B2];
    __shared__ __attribute__((aligned(1024))) uint16_t buf3[LD::B3];
    __shared__ __attribute__((aligned(1024))) uint16_t buf4[LD::B4];
    __shared__ __attribute__((aligned(1024))) uint16_t buf5[LD::B5];
    __shared__ __attribute__((aligned(1024))) uint16_t buf6[LD::B6];
    // gathered k rows' byte offsets in x (padded by two rings of stages; a
    // phased tile keeps them where its epilogue stages outputs)
    __shared__ uint32_t tok_s[LD::TOK];

    const int b = blockIdx.x;
    // column parts of a light expert's tiles: at most the expert's m-tile
    // slots of the grid (ceil(capacity / BM)), so the live tiles still fit it
    // (the d-wide row GEMMs: a few long tiles per expert; the f-wide ones have
    // many short light tiles already)
    using LT = typename LightOf<T>::type;
    constexpr bool LIGHT = light_ok<LT, A_KMAJOR, B_KMAJOR, EPI>();
    const int lsplit = LIGHT && (EPI == EPI_BIAS || EPI == EPI_STORE)
                           ? light_parts<LT>((batch.p[0].M + BM_ - 1) / BM_)
                           : 1;
    int qe = 0, qu = 0, qn = 0, qt = 0, qne = 0;  // quota: expert, rank, units, tiles, rows
    if constexpr (SCHED == 1) {
        // (in the first stage buffer, read before any stage is requested)
        static_assert(sizeof(QuotaPlan) <= sizeof(buf0), "the plan fits the buffer");
        QuotaPlan& qp = *reinterpret_cast<QuotaPlan*>(buf0);
        if (threadIdx.x < 64)
            build_quota_plan<EPI>(batch, BM_, lsplit, static_cast<int>(gridDim.x), &qp);
        __syncthreads();
        const int lane = threadIdx.x & 63;
        const int end = qp.first[lane] + qp.units[lane];
        const int e_b = __popcll(__ballot(end <= b));  // ends never decrease
        if (e_b >= batch.p[0].E) return;              // past every quota
        // (uniform values read from LDS: kept in scalar registers)
        qe = __builtin_amdgcn_readfirstlane(e_b);
        qn = __builtin_amdgcn_readfirstlane(qp.units[e_b]);
        qu = __builtin_amdgcn_readfirstlane(b - qp.first[e_b]);
        qt = __builtin_amdgcn_readfirstlane(qp.tiles[e_b]);
        qne = __builtin_amdgcn_readfirstlane(qp.ne[e_b]);
        __syncthreads();
    }
    for (int it = 0;; ++it) {
    int prob = 0, e, r, ne, tiles_m;
    if constexpr (SCHED == 1) {
        r = qu + it * qn;
        if (r >= qt) break;
        e = qe;
        ne = qne;
        if constexpr (compact_tiles<EPI>()) {
            tiles_m = expert_mtiles(ne, BM_, lsplit);
        } else {
            const int t0 = batch.tiles_m[0] * batch.tiles_n[0];
            prob = r >= t0 ? 1 : 0;
            if (prob) r -= t0;
            tiles_m = batch.tiles_m[prob];
        }
    } else {
    // Block b runs on XCD b mod 8 as that XCD's (b / 8)-th block; XCDs take
    // chunks of `chunk` consecutive tiles in turn, so the tiles resident on an
    // XCD share operand panels in its L2 while every XCD gets an even share of
    // each expert, however unevenly the rows are spread over experts.
    const int l = b >> 3, chunk = batch.chunk;
    int w = ((l / chunk) * 8 + (b & 7)) * chunk + l % chunk;
    if constexpr (EPI == EPI_BIAS || EPI == EPI_STORE) {
        const bool in = lsplit > 1
                            ? spread_tile(batch, BM_, lsplit, b & 7, l, 0, &e, &r, &ne)
                            : spread_tile(batch, BM_, lsplit, b & 7, (l / chunk) * 8 + (b & 7),
                                          l % chunk, &e, &r, &ne);
        if (!in) return;
        tiles_m = expert_mtiles(ne, BM_, lsplit);
    } else if constexpr (compact_tiles<EPI>()) {
        LiveTile lt;
        const GemmArgs& p0 = batch.p[0];
        if (!live_tile(p0.counts, p0.G, p0.E, p0.M, BM_, lsplit, batch.tiles_n[0], w, &lt)) return;
        e = lt.e;
        r = lt.r;
        ne = lt.ne;
        tiles_m = expert_mtiles(ne, BM_, lsplit);
    } else {
        if (w >= batch.total[0] + batch.total[1]) return;
        prob = w >= batch.total[0] ? 1 : 0;  // uniform per block
        if (prob) w -= batch.total[0];
        tiles_m = batch.tiles_m[prob];
        const int tiles_e = tiles_m * batch.tiles_n[prob];
        e = w / tiles_e;
        r = w - e * tiles_e;
        ne = expert_rows(batch.p[prob].counts, batch.p[prob].G, batch.p[prob].E, e);
    }
    }
    // (one value per block, kept in scalar registers)
    e = __builtin_amdgcn_readfirstlane(e);
    r = __builtin_amdgcn_readfirstlane(r);
    ne = __builtin_amdgcn_readfirstlane(ne);
    tiles_m = __builtin_amdgcn_readfirstlane(tiles_m);
    // The tile body, instantiated once per operand kind: with GS != 0 the
    // gathered operand is known at compile time, so a problem that gathers
    // and one that does not (the two weight gradients of one launch) each
    // get a main loop register-allocated for its own addressing alone.
    auto tile = [&](auto gather_kind) -> bool {
    constexpr int GS = decltype(gather_kind)::value;
    const GemmArgs& p = batch.p[prob];
    const int tiles_n = batch.tiles_n[prob];
    const int group_m = batch.group_m;
    // inside one expert, tiles go in groups of group_m m-tiles, m fastest, so
    // the blocks resident on an XCD at once cover a compact patch of the output
    // and share both operand panels in its L2
    const int grp = r / (group_m * tiles_n);
    const int first_m = grp * group_m;
    const int gm = min(group_m, tiles_m - first_m);
    const int idx = r - grp * group_m * tiles_n;
    const int tm = first_m + idx % gm;
    const int tn = idx / gm;
    const int rows = p.var_k ? p.M : min(ne, p.M);
    const int K = p.var_k ? ne : p.K;
    const int N = p.N;
    // An expert of two m-tiles has its rows split evenly (to whole 32-row
    // blocks): both stream the same weights, and a full tile beside one of a
    // few rows takes as long as the full one (288 rows an expert, 32 experts,
    // d = 1024, f = 4096: forward of the layer 309 -> 301 us)
    const int span = T::PHASED && !p.var_k && tiles_m == 2 && rows > BM_ ? (rows + 63) / 64 * 32
                                                                          : BM_;
    // a light expert's m-tile index is its column part
    const bool parts = lsplit > 1 && !p.var_k && ne > 0 && ne <= 32;
    const int m0 = parts ? 0 : tm * span, n0 = tn * BN_;
    if (m0 >= rows) return false;
    const int M = p.var_k ? rows : min(rows, m0 + span);

    static_assert(GS == 0 || (GS == 1 && A_KMAJOR) || (GS == 2 && !B_KMAJOR),
                  "gathered rows: k-major A or mn-major B");
    // gathered operands address x itself: its whole size is their range
    const __amdgpu_buffer_rsrc_t ra_rs =
        GS == 1 ? make_rsrc(p.a.base, p.gather_bytes)
           : make_rsrc(static_cast<const uint16_t*>(p.a.base) + e * p.a.estride,
                       p.a.estride * 2);
    const __amdgpu_buffer_rsrc_t rb_rs =
        GS == 2 ? make_rsrc(p.b.base, p.gather_bytes)
           : make_rsrc(static_cast<const uint16_t*>(p.b.base) + e * p.b.estride,
                       p.b.estride * 2);
    if constexpr (LIGHT) {
        if (!p.var_k && M - m0 <= 32) {
            light_tile<LT, GemmCfg<LT, EPI>, B_KMAJOR, EPI, GS>(
                p, ra_rs, rb_rs, e, M, N, K, m0, n0, parts ? tm : 0, parts ? lsplit : 1,
                LdsArrays{buf0, buf1, buf2, buf3, buf4, buf5, buf6});
            return true;
        }
    }
    if constexpr (T::PHASED) {
        phase_tile<T, A_KMAJOR, B_KMAJOR, EPI, GS>(p, ra_rs, rb_rs, e, M, N, K, m0, n0, tn, buf0,
                                                   buf1, buf2, buf3, buf4, buf5, buf6);
    } else {
        static_assert(!A_KMAJOR && !B_KMAJOR && EPI == EPI_F32, "small tiles: weight gradients");
        ring_tile<GS>(p, ra_rs, rb_rs, e, M, N, K, m0, n0, tn, buf0, buf1, buf2, buf3, tok_s);
    }
    return true;
    };
    bool ran;
    if constexpr (GATHER == 0) ran = tile(std::integral_constant<int, 0>{});
    else if (batch.p[prob].tok != nullptr) ran = tile(std::integral_constant<int, GATHER>{});
    else ran = tile(std::integral_constant<int, 0>{});
    if (!ran) {
        if constexpr (SCHED == 0) return;
        else continue;
    }
    if constexpr (SCHED == 0) break;
    // the next tile's first stages land in the buffers this epilogue staged
    // its outputs in: every wave's LDS accesses are done before any issues
    // them (its output stores stay in flight)
    lds_barrier();
    }
}

// ------------------------------------------------------------------ small batches

// Forward GEMMs of a layer whose expert buffers hold at most 32 RB rows (a few
// images served at a time): C[m, n] = sum_k A[m, k] B[n, k], both k-major, for
// all rows of one expert and 32 columns a block. Four waves split k in groups
// of 64, two groups in flight in registers, every load a coalesced 128-byte
// piece of a row; a group passes through LDS of the wave's own (16-byte
// chunks XOR-swizzled by row) to be read back as fragments. The waves' sums
// meet in LDS and are added in wave order, bias, GELU pair and rounding
// following in f32. Bound by latency: a launch of 256 x 256 tiles gives such a
// layer 24 to 96 CUs of work, each streaming up to 1.5 MB through one CU's
// share of the chip's bandwidth. (Fragments loaded straight from memory, 32
// rows an instruction, kept the address unit busy: 30 -> 46 us at 52 rows of
// 8 experts, d = 768, f = 3072, both GEMMs.)
template <int EPI, int RB, int GATHER>
__global__ __launch_bounds__(256) void small_rows_kernel(GemmArgs p) {
    static_assert(EPI == EPI_FWD1 || EPI == EPI_BIAS, "forward GEMMs");
    constexpr int NW = 4, ROWS = 32 * RB + 32;  // staged rows: A, then B
    constexpr int ST = ROWS * 64 * 2, PA = RB * 16 * 64 * 4;  // bytes per wave
    __shared__ __attribute__((aligned(16))) char lds[NW * (ST > PA ? ST : PA)];
    const int e = blockIdx.y, n0 = blockIdx.x * 32;
    const int ne = expert_rows(p.counts, p.G, p.E, e);
    const int M = min(ne, p.M), N = p.N, K = p.K;
    if (M == 0) return;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const __amdgpu_buffer_rsrc_t ra_rs =
        GATHER ? make_rsrc(p.a.base, p.gather_bytes)
               : make_rsrc(static_cast<const uint16_t*>(p.a.base) + e * p.a.estride,
                           p.a.estride * 2);
    const __amdgpu_buffer_rsrc_t rb_rs = make_rsrc(
        static_cast<const uint16_t*>(p.b.base) + e * p.b.estride, p.b.estride * 2);
    // load i of a group: row 8 i + lane / 8, elements 8 (lane % 8) .. + 7
    const int lr = lane >> 3, lc = 8 * (lane & 7);
    constexpr int LA = 4 * RB, LB = 4;
    int arow[LA], brow[LB];  // element offsets of the lane's rows, -1 outside
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int m = 8 * i + lr;
        arow[i] = m >= M ? -1 : (GATHER ? p.tok[e * p.tok_estride + m] : m) * p.a.ld;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int n = n0 + 8 * i + lr;
        brow[i] = n < N ? n * p.b.ld : -1;
    }
    const int ng = (K + 63) / 64;
    const int g0 = ng * wave / NW, g1 = ng * (wave + 1) / NW;
    uint4 fa[2][LA], fb[2][LB];
    auto load = [&](int u, int g) {  // (past the wave's last group nothing is read)
        const int k = 64 * g + lc;
        const bool in = g < g1 && k < K;
#pragma unroll
        for (int i = 0; i < LB; ++i)
            fb[u][i] = buf_load16(rb_rs, in && brow[i] >= 0 ? static_cast<uint32_t>(brow[i] + k) * 2u
                                                            : kOutOfRange);
#pragma unroll
        for (int i = 0; i < LA; ++i)
            fa[u][i] = buf_load16(ra_rs, in && arow[i] >= 0 ? static_cast<uint32_t>(arow[i] + k) * 2u
                                                            : kOutOfRange);
    };
    f32x16 acc[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[i][q] = 0.0f;
    uint16_t* const st = reinterpret_cast<uint16_t*>(lds + wave * ST);
    auto at = [&](int r, int c) { return st + r * 64 + ((c ^ (r & 7)) << 3); };
    load(0, g0);
    __builtin_amdgcn_sched_barrier(0);
    load(1, g0 + 1);
    __builtin_amdgcn_sched_barrier(0);
    for (int g = g0; g < g1; g += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            // (one wave's LDS accesses run in order: the previous group's reads
            // are done before these writes)
#pragma unroll
            for (int i = 0; i < LA; ++i)
                *reinterpret_cast<uint4*>(at(8 * i + lr, lane & 7)) = fa[u][i];
#pragma unroll
            for (int i = 0; i < LB; ++i)
                *reinterpret_cast<uint4*>(at(32 * RB + 8 * i + lr, lane & 7)) = fb[u][i];
            __builtin_amdgcn_sched_barrier(0);
            load(u, g + u + 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int c = 2 * s + (lane >> 5);
                const bf16x8 b =
                    *reinterpret_cast<const bf16x8*>(at(32 * RB + (lane & 31), c));
                // (swapped operands, as everywhere: lane l holds row l % 32)
#pragma unroll
                for (int i = 0; i < RB; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        b, *reinterpret_cast<const bf16x8*>(at(32 * i + (lane & 31), c)), acc[i],
                        0, 0, 0);
            }
        }
    }
    __syncthreads();  // every wave is done with its staged rows
    float* const part = reinterpret_cast<float*>(lds);  // [wave][i][register][lane]
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int q = 0; q < 16; ++q) part[((wave * RB + i) * 16 + q) * 64 + lane] = acc[i][q];
    __syncthreads();
    // wave w adds row blocks and columns 8 q + 4 (l / 32) + 0..3 of row l % 32
#pragma unroll
    for (int t = 0; t < RB; ++t) {
        const int i = t, q = wave;
        const int m = 32 * i + (lane & 31), n = n0 + 8 * q + 4 * (lane >> 5);
        if (m >= M || n >= N) continue;
        const uint2 bb = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(p.bias) +
                                                         e * p.bias_estride + n);
        float v[4] = {bf16_to_f32(bb.x & 0xFFFFu), bf16_to_f32(bb.x >> 16),
                      bf16_to_f32(bb.y & 0xFFFFu), bf16_to_f32(bb.y >> 16)};
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] += part[((w * RB + i) * 16 + 4 * q + c) * 64 + lane];
        const size_t o = e * p.out_estride + static_cast<size_t>(m) * p.ldo + n;
        if constexpr (EPI == EPI_FWD1) {
            float dg[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float h = v[c];
                gelu_pair(h, v[c], dg[c]);
            }
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out2) + o) =
                make_uint2(pack_bf16x2(dg[0], dg[1]), pack_bf16x2(dg[2], dg[3]));
        }
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + o) =
            make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    }
}

// ------------------------------------------------------------------ f32 path

// f32 activations: a block computes a 32 FB x 32 FB output tile of one expert
// with four waves that split k (whole runs of eight); every wave multiplies
// the whole tile over its share on v_mfma_f32_32x32x2_f32 (f32 products and
// sums), and the four partial tiles are added in wave order through LDS before
// the epilogue. A step is 32 deep. Of each eight k, lane l supplies row
// l % 32 and the four of half l / 32, in both operands. A k-major operand is
// read as 128-byte pieces of rows (16 bytes a lane) and passes through LDS of
// the wave's own, the next step's loads in flight meanwhile; an mn-major one is
// read straight into fragments, four coalesced dwords a run. No barrier stands
// before the partial tiles. Such a layer is bound by latency: the former
// 64 x 64 tiles of four waves side by side left the d-wide products of 788
// tokens (d = 192, f = 768, E = 8) on 96 blocks, each walking all 768 k behind
// two barriers a stage (30 and 36 us), and the bias gradients in two launches
// of 14 us, which the weight gradients' first n-tile now sums from its
// fragments. (k-major fragments straight from memory, 32 rows an instruction:
// forward 47 us against 50 before, 67 against 53 at d = 200, f = 800.) Layer step
// of the 788 tokens 216 -> 126 us, expert MLP forward 49 -> 28, backward
// 117 -> 54; 1576 tokens, k = 3, d = 384, f = 1536, E = 16: 199 -> 152, 437 -> 297.
// (Up-projections of a short k and very many tiles take 3 to 10 % longer than with
// the waves side by side, 4000 rows, E = 64, d = 64, f = 256 355 -> 399 us, and err
// two thirds to half as much: 9.7e-8 against 1.6e-7; with four sums a wave, to err
// the same, side by side takes 0.93 to 1.04 times the split's time.)
constexpr int kF32Waves = 4;
constexpr int kF32Ld = 32 + 4;  // LDS row: 32 k and 16 bytes (rows on other banks)

// k rows k .. k + 3 of one column of an mn-major operand, zero from kend (>= 1).
__device__ __forceinline__ float4 f32_cols(const float* col, int ld, int k, int kend) {
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        v[j] = col[static_cast<size_t>(min(k + j, kend - 1)) * ld];
    return make_float4(k < kend ? v[0] : 0.0f, k + 1 < kend ? v[1] : 0.0f,
                       k + 2 < kend ? v[2] : 0.0f, k + 3 < kend ? v[3] : 0.0f);
}

// One operand of a wave: 32 FB rows, a step in flight. Rows past `lim` read the
// last one (their outputs are never stored).
// (RUNS: runs of eight k a step, 4 where an operand is k-major).
template <bool KMAJOR, int FB, int RUNS>
struct F32Operand {
    static_assert(!KMAJOR || RUNS == 4, "128-byte row pieces");
    const float* p[KMAJOR ? 4 * FB : FB];
    float4 v[RUNS * FB];  // the step in flight
    int ld;
    __device__ __forceinline__ void init(const float* base, int ld_, int mn0, int lim, int lane) {
        ld = ld_;
        if constexpr (KMAJOR) {
#pragma unroll
            for (int i = 0; i < 4 * FB; ++i)
                p[i] = base + static_cast<size_t>(min(mn0 + 8 * i + (lane >> 3), lim - 1)) * ld +
                       4 * (lane & 7);
        } else {
#pragma unroll
            for (int i = 0; i < FB; ++i) p[i] = base + min(mn0 + 32 * i + (lane & 31), lim - 1);
        }
    }
    // request the step at k, zero from kend (a multiple of 8 for a k-major operand)
    __device__ __forceinline__ void load(int k, int kend, int lane) {
#pragma unroll
        for (int i = 0; i < RUNS * FB; ++i) {
            if constexpr (KMAJOR) {
                const bool in = k + 4 * (lane & 7) < kend;
                v[i] = *reinterpret_cast<const float4*>(p[i] + (in ? k : -4 * (lane & 7)));
                if (!in) v[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            } else {
                v[i] = f32_cols(p[i % FB], ld, k + 8 * (i / FB) + 4 * (lane >> 5), kend);
            }
        }
    }
    __device__ __forceinline__ void stage(float* s, int lane) const {
        if constexpr (KMAJOR) {
#pragma unroll
            for (int i = 0; i < 4 * FB; ++i)
                *reinterpret_cast<float4*>(s + (8 * i + (lane >> 3)) * kF32Ld + 4 * (lane & 7)) =
                    v[i];
        }
    }
    // run u's fragment of row block i: from LDS, or of the held step `h`
    __device__ __forceinline__ float4 frag(const float* s, const float4* h, int u, int i,
                                           int lane) const {
        if constexpr (KMAJOR)
            return *reinterpret_cast<const float4*>(s + (32 * i + (lane & 31)) * kF32Ld + 8 * u +
                                                    4 * (lane >> 5));
        else
            return h[u * FB + i];
    }
};

template <bool A_KMAJOR, bool B_KMAJOR, int EPI, int FB>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs p) {
    constexpr int FT = 32 * FB;
    // Two mn-major operands of 64 x 64 tiles: eight k a step, so that the
    // registers leave room for more waves
    constexpr int RUNS = !A_KMAJOR && !B_KMAJOR && FB == 2 ? 1 : 4;
    // a wave's staging of its k-major operands; afterwards the partial tiles
    constexpr int OP_EL = FT * kF32Ld, W_EL = ((A_KMAJOR ? 1 : 0) + (B_KMAJOR ? 1 : 0)) * OP_EL;
    constexpr int STG = kF32Waves * W_EL, PART = kF32Waves * 32 * FT;
    __shared__ __attribute__((aligned(16))) float lds[STG > PART ? STG : PART];
    __shared__ float rpart[EPI == EPI_F32 ? kF32Waves : 1][EPI == EPI_F32 ? FT : 1];
    float (*part)[32][FT] = reinterpret_cast<float (*)[32][FT]>(lds);
    const int e = blockIdx.z;
    const int ne = expert_rows(p.counts, p.G, p.E, e);
    const int M = p.var_k ? p.M : min(ne, p.M);
    const int K = p.var_k ? ne : p.K;
    const int N = p.N;
    const int m0 = blockIdx.y * FT, n0 = blockIdx.x * FT;
    if (m0 >= M) return;
    const int lane = threadIdx.x & 63, w = wave_id();
    const int r = lane & 31, kh = lane >> 5;
    // the wave's share of k, in runs of eight
    const int runs = (K + 7) / 8;
    const int k0 = 8 * (runs * w / kF32Waves);
    const int kend = min(K, 8 * (runs * (w + 1) / kF32Waves));
    const bool row_sum = EPI == EPI_F32 && p.bsum != nullptr && blockIdx.x == 0;
    float rs[FB];
    f32x16 acc[FB][FB];
#pragma unroll
    for (int i = 0; i < FB; ++i) {
        rs[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;
    }
    if (k0 < kend) {
        float* const as = lds + w * W_EL;
        float* const bs = as + (A_KMAJOR ? OP_EL : 0);
        F32Operand<A_KMAJOR, FB, RUNS> oa;
        F32Operand<B_KMAJOR, FB, RUNS> ob;
        oa.init(static_cast<const float*>(p.a.base) + e * p.a.estride, p.a.ld, m0, M, lane);
        ob.init(static_cast<const float*>(p.b.base) + e * p.b.estride, p.b.ld, n0, N, lane);
        oa.load(k0, kend, lane);
        ob.load(k0, kend, lane);
        for (int k = k0; k < kend; k += 8 * RUNS) {
            // (one wave's LDS accesses run in order: the last step's fragment
            // reads are done first)
            oa.stage(as, lane);
            ob.stage(bs, lane);
            float4 ha[A_KMAJOR ? 1 : RUNS * FB], hb[B_KMAJOR ? 1 : RUNS * FB];
            if constexpr (!A_KMAJOR) {
#pragma unroll
                for (int i = 0; i < RUNS * FB; ++i) ha[i] = oa.v[i];
            }
            if constexpr (!B_KMAJOR) {
#pragma unroll
                for (int i = 0; i < RUNS * FB; ++i) hb[i] = ob.v[i];
            }
            if (k + 8 * RUNS < kend) {
                oa.load(k + 8 * RUNS, kend, lane);
                ob.load(k + 8 * RUNS, kend, lane);
            }
#pragma unroll
            for (int u = 0; u < RUNS; ++u) {
                if (k + 8 * u >= kend) break;  // uniform
                float4 a[FB], b[FB];
#pragma unroll
                for (int i = 0; i < FB; ++i) {
                    a[i] = oa.frag(as, ha, u, i, lane);
                    b[i] = ob.frag(bs, hb, u, i, lane);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < FB; ++i) {
                        const float av = t == 0 ? a[i].x : t == 1 ? a[i].y : t == 2 ? a[i].z : a[i].w;
                        if constexpr (EPI == EPI_F32) rs[i] += av;
#pragma unroll
                        for (int j = 0; j < FB; ++j) {
                            const float bv =
                                t == 0 ? b[j].x : t == 1 ? b[j].y : t == 2 ? b[j].z : b[j].w;
                            acc[i][j] =
                                __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc[i][j], 0, 0, 0);
                        }
                    }
            }
        }
    }
    __syncthreads();  // every wave is past its staging: the partial tiles go there

    float* out = static_cast<float*>(p.out);
    const float* bias = static_cast<const float*>(p.bias);
    if constexpr (EPI == EPI_F32) {
        if (row_sum) {
#pragma unroll
            for (int i = 0; i < FB; ++i) {
                const float t = rs[i] + __shfl_xor(rs[i], 32, 64);
                if (lane < 32) rpart[w][32 * i + r] = t;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < FB; ++i) {
        if (i > 0) __syncthreads();
        // register q of lane l: row 8 (q / 4) + 4 (l / 32) + q % 4, column l % 32
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q)
                part[w][8 * (q / 4) + 4 * kh + (q % 4)][32 * j + r] = acc[i][j][q];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < FB; ++u) {
            const int v = u * 256 + static_cast<int>(threadIdx.x);
            const int row = v / (FT / 4), col = 4 * (v % (FT / 4));
            const int m = m0 + 32 * i + row, n = n0 + col;
            if (m >= M || n >= N) continue;
            float4 t = *reinterpret_cast<const float4*>(&part[0][row][col]);
            float x[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int w2 = 1; w2 < kF32Waves; ++w2) {
                t = *reinterpret_cast<const float4*>(&part[w2][row][col]);
                x[0] += t.x; x[1] += t.y; x[2] += t.z; x[3] += t.w;
            }
            const size_t o = e * p.out_estride + static_cast<size_t>(m) * p.ldo + n;
            if constexpr (EPI == EPI_FWD1 || EPI == EPI_BIAS) {
                t = *reinterpret_cast<const float4*>(bias + e * p.bias_estride + n);
                x[0] += t.x; x[1] += t.y; x[2] += t.z; x[3] += t.w;
            }
            if constexpr (EPI == EPI_GELU_GRAD) {
                t = *reinterpret_cast<const float4*>(static_cast<const float*>(p.aux) + o);
                x[0] *= t.x; x[1] *= t.y; x[2] *= t.z; x[3] *= t.w;
            }
            if constexpr (EPI == EPI_FWD1) {
                *reinterpret_cast<float4*>(static_cast<float*>(p.out2) + o) =
                    make_float4(gelu_grad_f(x[0]), gelu_grad_f(x[1]), gelu_grad_f(x[2]),
                                gelu_grad_f(x[3]));
#pragma unroll
                for (int c = 0; c < 4; ++c) x[c] = gelu_f(x[c]);
            }
            // (weight gradients: streaming stores, as on the bf16 path; backward
            // at 64 rows, E = 32, d = 1024, f = 4096 1060 -> 1017 us)
            const float4 y = make_float4(x[0], x[1], x[2], x[3]);
            if constexpr (EPI == EPI_F32)
                __builtin_nontemporal_store(__builtin_bit_cast(v4i32, y),
                                            reinterpret_cast<v4i32*>(out + o));
            else
                *reinterpret_cast<float4*>(out + o) = y;
        }
        if constexpr (EPI == EPI_F32) {
            const int t = threadIdx.x;
            if (row_sum && i == 0 && t < FT && m0 + t < M)
                p.bsum[static_cast<size_t>(e) * M + m0 + t] =
                    ((rpart[0][t] + rpart[1][t]) + rpart[2][t]) + rpart[3][t];
        }
    }
}

constexpr int kNumCUs = 256;

// One launch over `n` (1 or 2) problems; grid_m_rows[i] bounds problem i's m.
template <class T, bool AK, bool BK_, int EPI, int GATHER = 0>
void launch_bf16(const Dims& D, const GemmArgs* a, const int* grid_m_rows, int n, int sched,
                 hipStream_t st) {
    GemmBatch b{};
    for (int i = 0; i < n; ++i) {
        b.p[i] = a[i];
        b.tiles_m[i] = static_cast<int>(cdiv(grid_m_rows[i], T::BM));
        b.tiles_n[i] = static_cast<int>(cdiv(a[i].N, T::BN));
        b.total[i] = D.E * b.tiles_m[i] * b.tiles_n[i];
    }
    // blocks resident on one XCD: 32 CUs x blocks per CU. A single problem
    // with both operands k-major whose experts span at most 8 m-tiles is
    // dealt a whole m-column of one expert per chunk (each XCD streams one
    // expert's row panels past four of its weight panels; measured faster for
    // the forward GEMMs, slower for the transposed-weight ones); otherwise
    // patches of 4 m-tiles.
    const int one_col = AK && BK_ && n == 1 && b.tiles_m[0] <= 8 ? b.tiles_m[0] : 0;
    b.group_m = one_col ? one_col : (T::WAVES_PER_EU == 2 && T::NW == 4 ? 8 : 4);
    b.chunk = 4 * b.group_m;
    // (the spread row GEMMs take one chunk more per XCD: splitting the tiles
    // into two classes can leave a partial chunk in each)
    const int spread = EPI == EPI_BIAS || EPI == EPI_STORE ? 1 : 0;
    b.per_xcd = static_cast<int>(cdiv(b.total[0] + b.total[1], 8 * b.chunk) + spread) * b.chunk;
    if (sched && GATHER == 0) {
        // persistent blocks under quotas: as many as are resident at once
        // (one per CU for the 8-wave tiles, two for the 4-wave ones)
        const int resident = kNumCUs * (T::NW == 8 ? 1 : T::WAVES_PER_EU);
        const int grid = min(8 * b.per_xcd, resident);
        gemm_bf16_kernel<T, AK, BK_, EPI, 1><<<grid, T::NT, 0, st>>>(b);
    } else {
        gemm_bf16_kernel<T, AK, BK_, EPI, 0, GATHER><<<8 * b.per_xcd, T::NT, 0, st>>>(b);
    }
}

template <class T, bool AK, bool BK_, int EPI, int GATHER = 0>
void launch_bf16(const Dims& D, const GemmArgs& a, int grid_m_rows, int sched, hipStream_t st) {
    launch_bf16<T, AK, BK_, EPI, GATHER>(D, &a, &grid_m_rows, 1, sched, st);
}

// Tilings: 256 x 256 and 256 x 192 (fewer idle CUs where an output is d wide),
// beside SmallTile.
using TileBig = PhaseTile<4>;
using TileNarrow = PhaseTile<3>;

// Relative cost per tile area of the other tilings (256 x 256 is 1): of the
// factors 1.0 to 1.6 for 128 x 128 and 1.0 to 1.15 for 256 x 192, those whose choice
// came closest to the fastest tiling of each of 313 expert MLP backwards (d = 192
// to 1024, f = 2 d to 4 d, E = 4 to 64, 16 to 1000 rows): 1.4 % above it in the mean.
// (1.15 for 128 x 128, from the time before the 256-row tiles were phased, was
// 3.3 % above it: 1000 rows, E = 32, d = 776, f = 3104 1061 us against 864, the
// 128 x 128 tiles also holding up dxe beside them; 150 rows, E = 24, d = 384,
// f = 1536 89 against 71.)
constexpr double kNarrowCost = 1.05;
constexpr double kSmallCost = 1.3;

// Work of a launch in units of one CU's time: rounds of one-block-per-CU
// waves times the tile's area (relative cost per tile area `eff`).
double tile_cost(long long tiles, int bm, int bn, double eff) {
    return static_cast<double>((tiles + kNumCUs - 1) / kNumCUs) * bm * bn * eff;
}

template <bool AK, bool BK_, int EPI, int GATHER = 0>
void launch_gemm(const Dims& D, const GemmArgs& a, int grid_m_rows, int sched, hipStream_t st) {
    // Few rows an expert, and so few tiles that a quarter of the CUs or more
    // would have none: small code over many blocks instead. Expert MLP forward
    // at d = 768, f = 3072, 52 rows: E = 8 (96 and 32 tiles) 48.5 -> 29.5 us,
    // E = 12 50.8 -> 45.3, E = 16 (192 and 64 tiles) 52.0 -> 49.9, E = 32 even;
    // E = 64 at d = 512, f = 2048 slower (80 -> 93), and with 103 rows at
    // E = 8 too (51 -> 54: the blocks read an expert's rows over and over).
    // (Independent of `sched`: an expert is one tile, there is nothing to share.)
    if constexpr (EPI == EPI_FWD1 || EPI == EPI_BIAS) {
        if (D.dtype == VMOE_BF16 && grid_m_rows <= 64 &&
            static_cast<long long>(D.E) * cdiv(a.N, 256) <= kNumCUs * 3 / 4) {
            const dim3 grid(cdiv(a.N, 32), D.E);
            if (grid_m_rows <= 32)
                small_rows_kernel<EPI, 1, GATHER><<<grid, 256, 0, st>>>(a);
            else
                small_rows_kernel<EPI, 2, GATHER><<<grid, 256, 0, st>>>(a);
            return;
        }
    }
    // (bf16 weight gradients run batched in ffn_bwd_launch)
    if constexpr (EPI != EPI_F32) {
        if (D.dtype == VMOE_BF16) {
            // 256 x 256 tiles (half the operand bytes per flop of 128 x 128). Outputs
            // N = d_model wide give few tiles: 192-column tiles fill more CUs when
            // that saves a round. (The f-wide outputs have tiles enough; with
            // 256 x 192 there too the ViT-B/16 expert MLP forward took 162 -> 168 us,
            // the 17-task step 1211 -> 1231, eight ViT-L/16 images 294 -> 311.)
            if constexpr (EPI == EPI_BIAS || EPI == EPI_STORE) {
                const long long tm = cdiv(grid_m_rows, 256);
                const double big = tile_cost(D.E * tm * cdiv(a.N, 256), 256, 256, 1.0);
                const double narrow = tile_cost(D.E * tm * cdiv(a.N, 192), 256, 192, kNarrowCost);
                if (narrow < big) {
                    launch_bf16<TileNarrow, AK, BK_, EPI, GATHER>(D, a, grid_m_rows, sched, st);
                    return;
                }
            }
            launch_bf16<TileBig, AK, BK_, EPI, GATHER>(D, a, grid_m_rows, sched, st);
            return;
        }
    }
    // 64 x 64 tiles halve the operand loads a product, 32 x 32 ones give a
    // launch four times the blocks and the waves more registers: with 64
    // from three blocks a CU on for the weight gradients (two mn-major
    // operands; backward at 400 tokens, d = 256, f = 1024, E = 16: 55 us
    // against 61 with 32) and from twelve on for the others (from three on:
    // forward 101 -> 111, backward 227 -> 236 at 1576 tokens, d = 384,
    // f = 1536, E = 8)
    const long long big = static_cast<long long>(D.E) * cdiv(grid_m_rows, 64) * cdiv(a.N, 64);
    if (big >= kNumCUs * (EPI == EPI_F32 ? 3 : 12)) {
        const dim3 grid(cdiv(a.N, 64), cdiv(grid_m_rows, 64), D.E);
        gemm_f32_kernel<AK, BK_, EPI, 2><<<grid, 256, 0, st>>>(a);
    } else {
        const dim3 grid(cdiv(a.N, 32), cdiv(grid_m_rows, 32), D.E);
        gemm_f32_kernel<AK, BK_, EPI, 1><<<grid, 256, 0, st>>>(a);
    }
}

GemmArgs base_args(const Dims& D, const int32_t* counts) {
    GemmArgs a{};
    a.counts = counts;
    a.G = D.G;
    a.E = D.E;
    return a;
}

// A second stream per GPU (default priority, non-blocking) and two events,
// made on first use, for launches that may run beside the caller's stream:
// the caller's stream records `fork`, the side stream waits for it, takes
// its launches and records `join`, which the caller's stream waits for, so
// the call still completes in its stream's order (and a captured stream
// captures the side stream's work as a branch of its graph).
struct SideStream {
    hipStream_t s = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
};
constexpr int kMaxSideDevices = 64;
std::mutex side_mu;
SideStream side_tab[kMaxSideDevices];
// held by a call from its fork to its join, so calls from several host
// threads never interleave their event records and waits
std::mutex side_seq_mu;

// The current GPU's side stream, or null fields on a HIP error (the caller
// then runs everything on its own stream).
SideStream side_stream() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxSideDevices) return {};
    std::lock_guard<std::mutex> lock(side_mu);
    SideStream& t = side_tab[dev];
    if (t.s == nullptr) {
        SideStream n;
        if (hipStreamCreateWithFlags(&n.s, hipStreamNonBlocking) != hipSuccess) return {};
        if (hipEventCreateWithFlags(&n.fork, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&n.join, hipEventDisableTiming) != hipSuccess) {
            if (n.fork) (void)hipEventDestroy(n.fork);
            (void)hipStreamDestroy(n.s);
            return {};
        }
        t = n;
    }
    return t;
}

// One wave: the device fill-clamp-refill of n experts (the routine the
// quota-scheduled GEMMs run), for comparison with the host routine.
__global__ __launch_bounds__(64) void fcr_kernel(int n, const int32_t* __restrict__ mn,
                                                 const int32_t* __restrict__ sat,
                                                 const double* __restrict__ coef, int budget,
                                                 int32_t* __restrict__ units) {
    const int lane = threadIdx.x;
    const int u = fill_clamp_refill_wave(n, lane < n ? mn[lane] : 0, lane < n ? sat[lane] : 0,
                                         lane < n ? coef[lane] : 0.0, budget);
    if (lane < n) units[lane] = u;
}

}  // namespace

vmoe_status fcr_device_launch(int n, const int32_t* mn, const int32_t* sat, const double* coef,
                              int budget, int32_t* units, hipStream_t st) {
    if (n > 0) fcr_kernel<<<1, 64, 0, st>>>(n, mn, sat, coef, budget, units);
    return launch_status();
}

vmoe_status ffn_fwd_launch(const Dims& D, const void* xe, const int32_t* counts, const void* w1,
                           const void* b1, const void* w2, const void* b2, void* act,
                           void* act_grad, void* ye, int sched, const int32_t* row_token,
                           hipStream_t st) {
    const long long rows = D.rows_per_expert();
    if (rows == 0 || D.E == 0) return VMOE_OK;
    // H = xe W1^T + b1 (never stored), A = gelu(H), A' = gelu'(H)
    GemmArgs g1 = base_args(D, counts);
    g1.a = Operand{xe, rows * D.d, D.d};
    g1.b = Operand{w1, static_cast<long long>(D.f) * D.d, D.d};
    g1.M = static_cast<int>(rows);
    g1.N = D.f;
    g1.K = D.d;
    g1.out = act;
    g1.out2 = act_grad;
    g1.out_estride = rows * D.f;
    g1.ldo = D.f;
    g1.bias = b1;
    g1.bias_estride = D.f;
    if (row_token != nullptr) {
        // dispatch fused into the loads: row r of expert e is x[row_token[e, r]]
        g1.a = Operand{xe, 0, D.d};
        g1.tok = row_token;
        g1.tok_estride = rows;
        g1.gather_bytes = static_cast<long long>(D.N) * D.d * 2;
        launch_gemm<true, true, EPI_FWD1, 1>(D, g1, static_cast<int>(rows), sched, st);
    } else {
        launch_gemm<true, true, EPI_FWD1>(D, g1, static_cast<int>(rows), sched, st);
    }
    // ye = A W2^T + b2
    GemmArgs g2 = base_args(D, counts);
    g2.a = Operand{act, rows * D.f, D.f};
    g2.b = Operand{w2, static_cast<long long>(D.d) * D.f, D.f};
    g2.M = static_cast<int>(rows);
    g2.N = D.d;
    g2.K = D.f;
    g2.out = ye;
    g2.out_estride = rows * D.d;
    g2.ldo = D.d;
    g2.bias = b2;
    g2.bias_estride = D.d;
    launch_gemm<true, true, EPI_BIAS>(D, g2, static_cast<int>(rows), sched, st);
    return launch_status();
}

vmoe_status ffn_bwd_launch(const Dims& D, const void* xe, const int32_t* counts, const void* w1,
                           const void* w2, const void* act, const void* act_grad, const void* dye,
                           void* dh, void* dxe, float* dw1, float* db1, float* dw2, float* db2,
                           int sched, const int32_t* row_token, hipStream_t st) {
    const long long rows = D.rows_per_expert();
    if (D.E == 0) return VMOE_OK;
    SideStream side;  // set when dxe runs beside the weight gradients
    std::unique_lock<std::mutex> seq;
    if (rows > 0) {
        // dH = (dye W2) * A': W2 [d, f] read with k = d strided (mn-major)
        GemmArgs g = base_args(D, counts);
        g.a = Operand{dye, rows * D.d, D.d};
        g.b = Operand{w2, static_cast<long long>(D.d) * D.f, D.f};
        g.M = static_cast<int>(rows);
        g.N = D.f;
        g.K = D.d;
        g.out = dh;
        g.out_estride = rows * D.f;
        g.ldo = D.f;
        g.aux = act_grad;
        launch_gemm<true, false, EPI_GELU_GRAD>(D, g, static_cast<int>(rows), sched, st);
        // dxe = dH W1: W1 [f, d] read with k = f strided
        GemmArgs x = base_args(D, counts);
        x.a = Operand{dh, rows * D.f, D.f};
        x.b = Operand{w1, static_cast<long long>(D.f) * D.d, D.d};
        x.M = static_cast<int>(rows);
        x.N = D.d;
        x.K = D.f;
        x.out = dxe;
        x.out_estride = rows * D.d;
        x.ldo = D.d;
        // dxe and the weight gradients both read only dH and the layer's saved
        // tensors: dxe runs on the side stream beside them, so the weight-
        // gradient blocks take the CUs that its partly filled tiles and last
        // round leave idle (bf16, one-tile-per-block schedule, 16 or more
        // experts: 17-task step 1254 -> 1213 us, expert-MLP backward of the wide
        // E = 32 pool 1041 -> 1019; with 8 evenly loaded experts every tile is
        // full and the two launches only contend, ViT-B/16 step 523 -> 532)
        if (D.dtype == VMOE_BF16 && sched == 0 && D.E >= 16) {
            seq = std::unique_lock<std::mutex>(side_seq_mu);
            side = side_stream();
            if (side.s != nullptr && (hipEventRecord(side.fork, st) != hipSuccess ||
                                      hipStreamWaitEvent(side.s, side.fork, 0) != hipSuccess))
                side = SideStream{};
        }
        launch_gemm<true, false, EPI_STORE>(D, x, static_cast<int>(rows), sched,
                                            side.s != nullptr ? side.s : st);
    }
    // dW2 [d, f] = dye^T A, reduced over the n_e rows (k = row, strided)
    GemmArgs w = base_args(D, counts);
    w.var_k = 1;
    w.a = Operand{dye, rows * D.d, D.d};
    w.b = Operand{act, rows * D.f, D.f};
    w.M = D.d;
    w.N = D.f;
    w.K = 0;
    w.out = dw2;
    w.out_estride = static_cast<long long>(D.d) * D.f;
    w.ldo = D.f;
    w.bsum = db2;  // db2 = row sums of dye^T
    // dW1 [f, d] = dH^T xe
    GemmArgs v = base_args(D, counts);
    v.var_k = 1;
    v.a = Operand{dh, rows * D.f, D.f};
    v.b = Operand{xe, rows * D.d, D.d};
    v.M = D.f;
    v.N = D.d;
    v.K = 0;
    v.out = dw1;
    v.out_estride = static_cast<long long>(D.f) * D.d;
    v.ldo = D.d;
    v.bsum = db1;  // db1 = row sums of dH^T
    if (row_token != nullptr) {
        // xe rows gathered from x: row r of expert e is x[row_token[e, r]]
        v.b = Operand{xe, 0, D.d};
        v.tok = row_token;
        v.tok_estride = rows;
        v.gather_bytes = static_cast<long long>(D.N) * D.d * 2;
    }
    if (D.dtype == VMOE_BF16) {
        // both weight gradients in one launch (same kernel, independent tiles),
        // with the tiling of the least cost in rounds x tile area (128 x 128
        // tiles run two per CU and cost more per flop)
        const GemmArgs both[2] = {w, v};
        const int rows_m[2] = {D.d, D.f};
        auto tiles = [&](int bm, int bn) {
            return D.E * (static_cast<long long>(cdiv(D.d, bm)) * cdiv(D.f, bn) +
                          static_cast<long long>(cdiv(D.f, bm)) * cdiv(D.d, bn));
        };
        const double small = tile_cost((tiles(128, 128) + 1) / 2, 256, 128, kSmallCost);
        const double narrow = tile_cost(tiles(256, 192), 256, 192, kNarrowCost);
        const double big = tile_cost(tiles(256, 256), 256, 256, 1.0);
        // (the gathered input-weight gradient takes the same tiling, so its
        // results, bias-gradient sums included, are the unfused call's bits)
        auto go = [&](auto gather) {
            constexpr int GA = decltype(gather)::value;
            if (narrow <= small && narrow <= big)
                launch_bf16<TileNarrow, false, false, EPI_F32, GA>(D, both, rows_m, 2, sched, st);
            else if (big <= small)
                launch_bf16<TileBig, false, false, EPI_F32, GA>(D, both, rows_m, 2, sched, st);
            else
                launch_bf16<SmallTile, false, false, EPI_F32, GA>(D, both, rows_m, 2, sched, st);
        };
        if (row_token != nullptr) go(std::integral_constant<int, 2>{});
        else go(std::integral_constant<int, 0>{});
    } else {
        launch_gemm<false, false, EPI_F32>(D, w, D.d, 0, st);
        launch_gemm<false, false, EPI_F32>(D, v, D.f, 0, st);
    }
    if (side.s != nullptr) {
        // the call ends in its stream's order: after the side stream's dxe
        const vmoe_status ls = launch_status();
        if (hipEventRecord(side.join, side.s) != hipSuccess ||
            hipStreamWaitEvent(st, side.join, 0) != hipSuccess)
            return VMOE_ERR_HIP;
        if (ls != VMOE_OK) return ls;
    }
    return launch_status();
}

}  // namespace vmoe
