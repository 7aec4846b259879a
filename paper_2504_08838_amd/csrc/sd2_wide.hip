// libsd2 -- linears on 17 to 64 tokens (gfx950): bitmask, 2:4 and dense matrices in one kernel.
//
// What bounds a wide call is not the matrix stream but the activations: 64 tokens x 3072 columns are 393 KB, more than a
// compute unit's LDS and three quarters of its registers, so a kernel that streams the matrix once and walks the whole
// contraction strip by strip fetches the activations again for every tile (1 KB of them per 64 bytes of matrix).  Here
// the activations stay and the strips pass by: a wavefront holds the activations of one unit of 128 columns
// (16 registers per 16 tokens) and the running sums of SG strips (up to 64 registers); a pass takes the unit's part of
// each of the strips -- expanded from the bitmask, or loaded as it is, once for all tokens -- and the next pass takes the
// next unit.  Nothing synchronises the wavefronts until the strips are complete; then the sums of the wavefronts that
// shared the contraction meet in LDS, are added in a fixed order and leave as final values (or, [gate; up], as the
// gated product).  (A first version with twelve wavefronts met in LDS after every strip and unit: the 3B shape's gate|up
// on 64 tokens took 28 us, nearly twice the expansion's own time, all wavefronts waiting out each other's latencies.)
//
// A matrix with few strips has its contraction split over workgroups as well; each leaves a partial result that the next
// kernel adds.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "sd2_device.h"
#include "sd2_format.h"
#include "sd2_internal.h"

namespace sd2 {

typedef __attribute__((__vector_size__(16 * sizeof(__bf16)))) __bf16 bf16x16;
union Frag16 {
    u32x4 q[2];
    bf16x16 v;
};

// Where a workgroup's work lies.  Workgroup b takes split b % n_split of the contraction and strip block b / n_split.
struct WideArgs {
    const uint8_t* dir;    // directory (bitmask)
    const uint8_t* masks;
    const uint8_t* vals;
    const uint8_t* tiles;  // 2:4
    const uint16_t* w;     // dense
    const uint16_t* x;
    float* out;            // [n_split][k_tok][n_out], or bf16 [k_tok][n_out / 2] (gated)
    int n_out, k_in, k_tok, n_strips;
    int n_units;           // ceil(k_in / 128)
    int n_split, n_pass;   // splits of the contraction over workgroups; passes of a workgroup over its strips
    int wk;                // wavefronts along the contraction (even); the other ways split the strips of a group
    int strips_per_wg;     // strips a workgroup owns
    int half_strips;       // gated: strips of one half of [gate; up], whose strips alternate; else 0
};

enum { kWideBitmask = 0, kWideNm24 = 1, kWideDense = 2 };

template <int FMT>
struct WideStage;  // two 64-column steps of one strip on their way from memory
template <>
struct WideStage<kWideBitmask> {  // 2560 bytes of the stream in registers (enough down to 40 % sparsity; the rest is fetched late)
    u32x4 v[2];
    uint2 tail;
    uint32_t mk;
};
template <>
struct WideStage<kWideNm24> {
    u32x4 v[2];
    uint32_t idx;
};
template <>
struct WideStage<kWideDense> {
    u32x4 v[4];
};
constexpr uint32_t kWideStaged = 2560;

// A wavefront's LDS: the staged stream of half a tile (it can hold 4096 bytes of values when a tile's values crowd into one
// half, 14 bytes of misalignment and 8 of slack), or a block that goes from row order to operand order.
constexpr int kWideBufDw = (4096 + 32) / 4;

// Where the wavefronts' sums meet when a group's strips are complete.  Behind the buffers no wavefront waits for the others' last
// reads before it leaves its sums, but that needs room: four strips of four token groups take the buffers' place.
constexpr size_t wide_sums_bytes(int sg, int tg, int w) { return (size_t)sg * w * tg * 1024; }
constexpr bool wide_apart(int sg, int tg, int w) { return wide_sums_bytes(sg, tg, w) + (size_t)w * kWideBufDw * 4 <= 159 * 1024; }

// One 64-column step of a bitmask tile between its LDS reads and their use: the windows of its four runs, their selectors and
// byte offsets.  The reads of a step are issued before the step ahead of it is used, so that a wavefront always has LDS
// reads in flight while it works (two wavefronts on a SIMD do not hide each other's LDS round trips).
struct WideWindow {
    Tri32 tr[4];
    uint2 sel[4];
    uint32_t off[4];
};

// exclusive prefix counts of the nibbles of two steps (mask word m), four bytes each
__device__ __forceinline__ void wide_scan(uint32_t m, uint32_t (&ex)[2]) {
    uint32_t x = m - ((m >> 1) & 0x55555555u);
    x = (x & 0x33333333u) + ((x >> 2) & 0x33333333u);
    const uint32_t even = x & 0x0f0f0f0fu, odd = (x >> 4) & 0x0f0f0f0fu;
    ex[0] = __builtin_amdgcn_perm(odd, even, 0x05010400u);
    ex[1] = __builtin_amdgcn_perm(odd, even, 0x07030602u);
    wave_excl_scans(ex);
}

// lane0: the lane of `runs` that holds the LDS byte address of the step's first run; m16: the step's mask
__device__ __forceinline__ void wide_reads(WideWindow& w, uint32_t runs, int lane0, const uint2* __restrict__ lut, uint32_t ex, uint32_t m16) {
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        w.off[h] = (uint32_t)__builtin_amdgcn_readlane((int)runs, lane0 + h) + __builtin_amdgcn_ubfe(ex, 8 * h, 8) * 2u;
        const __attribute__((address_space(3))) uint32_t* win = (const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(w.off[h] & ~3u);
        w.tr[h].a = win[0];
        w.tr[h].b = win[1];
        w.tr[h].c = win[2];
        w.sel[h] = lut[__builtin_amdgcn_ubfe(m16, 4 * h, 4)];
    }
}

__device__ __forceinline__ void wide_fragments(const WideWindow& w, Frag& f0, Frag& f1) {
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const uint32_t w0 = __builtin_amdgcn_alignbyte(w.tr[h].b, w.tr[h].a, w.off[h]);
        const uint32_t w1 = __builtin_amdgcn_alignbyte(w.tr[h].c, w.tr[h].b, w.off[h]);
        Frag& f = h < 2 ? f0 : f1;
        f.u[2 * (h & 1) + 0] = __builtin_amdgcn_perm(w1, w0, w.sel[h].x);
        f.u[2 * (h & 1) + 1] = __builtin_amdgcn_perm(w1, w0, w.sel[h].y);
    }
}

// A block of 16 rows x 128 columns (256 bytes a row) of a row-major bf16 matrix.  Loaded row by row -- sixteen consecutive lanes
// take one row, so that a load touches eight cache lines; a lane per row would touch 64 --
// `p` is the block's first element; rows past last_row repeat it, columns past n_cols repeat the block's first column.
__device__ __forceinline__ u32x4 block_piece(const uint16_t* p, uint32_t row, uint32_t last_row, uint32_t n_cols, uint32_t k_in, int lane) {
    const uint32_t r = min(row + (uint32_t)(lane >> 4), last_row), c = 8u * (uint32_t)(lane & 15);
    return *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(p) + (r * k_in + (c < n_cols ? c : 0u)) * 2u);
}
// and turned through the wavefront's own LDS into matrix operands (lane = row n, columns 64 q + 16 g + 8 e: entry 2 q + e).  Piece
// j of row r sits at piece j ^ r: both directions touch every bank once.
__device__ __forceinline__ void block_to_operands(u32x4 (&v)[4], uint32_t* buf, int lane) {
    u32x4* b16 = reinterpret_cast<u32x4*>(buf);
    const int n = lane & 15, g = lane >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 4 * i + g;
        b16[r * 16 + (n ^ r)] = v[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = b16[n * 16 + ((8 * (i >> 1) + 2 * g + (i & 1)) ^ n)];
}

__device__ __forceinline__ uint32_t wide_lane(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }

#define SD2_INLINE __attribute__((always_inline))

template <int FMT, int TG, int SG, int W>
__global__ __launch_bounds__(64 * W) void wide_linear_kernel(const WideArgs a) {
    constexpr bool kAhead = W == 8 ? TG * SG < 16 : TG * SG <= 4;  // LDS reads of a step ahead of the use of the one before it
    typedef WideStage<FMT> Stage;
    extern __shared__ __attribute__((aligned(16))) uint32_t wide_smem[];
    __shared__ uint2 lut[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    if (FMT == kWideBitmask) {
        if (tid < 16) lut[tid] = make_expand_selector((uint32_t)tid);
        __syncthreads();
    }
    uint32_t* buf = wide_smem + wave * kWideBufDw;
    // sums of the wavefronts [strip of the group][wk][TG][256]: behind the buffers where both fit, else in their place
    constexpr bool kApart = wide_apart(SG, TG, W);
    float* red = reinterpret_cast<float*>(wide_smem) + (kApart ? W * kWideBufDw : 0);

    const int split = (int)blockIdx.x % a.n_split, sblk = (int)blockIdx.x / a.n_split;
    const int n_pass = a.n_pass, wk = a.wk, ws = W / wk;
    const int sw = wave / wk, kw = wave - sw * wk;
    const int s0 = sblk * a.strips_per_wg;
    const int my_strips = min(a.strips_per_wg, a.n_strips - s0);
    const int group = SG * ws;
    const int n_grp = (my_strips + group - 1) / group, n_rounds = n_grp * n_pass;
    const int unit0 = split * n_pass * wk + kw;  // unit of pass p: unit0 + p * wk
    const int my_half = kw & 1;                  // the half of a tile that this wavefront takes (wk is even)
    // strips of the workgroup in order: s0, s0 + 1, ... -- or, gated, gate strip p and up strip half + p of pair p in turn
    const bool gated = a.half_strips != 0;
    auto strip_of = [&](int ord) SD2_INLINE { return gated ? (s0 >> 1) + (ord >> 1) + (ord & 1) * a.half_strips : s0 + ord; };

    // a round: one pass over one group of strips; scalar arithmetic without branches
    struct Round {
        int grp, pass;
    };
    auto next = [&](const Round& r) SD2_INLINE {
        const int pass = r.pass + 1, over = pass == n_pass ? 1 : 0;
        return Round{r.grp + over, over ? 0 : pass};
    };
    auto unit_at = [&](const Round& r) SD2_INLINE { return unit0 + r.pass * wk; };
    auto ord_at = [&](const Round& r, int i) SD2_INLINE { return r.grp * group + sw * SG + i; };
    auto live = [&](const Round& r, int i) SD2_INLINE {
        return ((int)(r.grp < n_grp) & (int)(ord_at(r, i) < my_strips) & (int)(unit_at(r) < a.n_units)) != 0;
    };
    // tile of the wavefront's strip i in a round; one that does not exist reads tile 0, and is not used
    auto tile_at = [&](const Round& r, int i) SD2_INLINE {
        const uint32_t t = (uint32_t)(unit_at(r) >> 1) * (uint32_t)a.n_strips + (uint32_t)strip_of(ord_at(r, i));
        return live(r, i) ? t : 0u;
    };

    // Every load whose wait the compiler counts is issued on every path: a request that may or may not have happened makes
    // it wait for everything in flight.

    // What a round needs of its tiles, in lanes: the sixteen lanes 16 i .. 16 i + 15 belong to strip i.  A few vector
    // operations per round take the place of scalar arithmetic per tile (with two wavefronts on a SIMD every instruction
    // counts, scalar ones too); a tile's numbers are picked with v_readlane.
    struct Tiles {
        uint32_t t;        // tile
        uint2 head;        // bitmask: val_start, nnz ...
        uint32_t mid;      // ... values before the second half
        uint32_t run;      // ... values before run (lane & 7) of the wavefront's half
    };
    auto directory = [&](const Round& r) SD2_INLINE {
        Tiles d;
        uint32_t t = 0u;
#pragma unroll
        for (int i = 0; i < SG; ++i) {
            const uint32_t ti = tile_at(r, i);
            t = (lane >> 4) == i ? ti : t;
        }
        d.t = t;
        if (FMT == kWideBitmask) {
            const uint8_t* e = a.dir + (size_t)t * 48;
            d.head = *reinterpret_cast<const uint2*>(e);
            d.mid = *reinterpret_cast<const uint16_t*>(e + 24);
            d.run = *reinterpret_cast<const uint16_t*>(e + 8 + 2 * (8 * my_half + (lane & 7)));
        }
        return d;
    };
    // the part of a tile's stream that the wavefront's half takes: 16 n16 bytes from `off`, a byte offset into the value
    // section (32 bits, checked by the host); the first of them is byte `lo` of the tile's stream (a multiple of 16)
    struct Parts {
        uint32_t off, n16, lo;
    };
    auto parts_of = [&](const Tiles& d) SD2_INLINE {
        Parts p;
        const uint32_t second = 0u - (uint32_t)my_half, mid = d.mid * 2u, all = d.head.y * 2u;
        p.lo = mid & ~15u & second;
        p.n16 = (((all & second) | (mid & ~second)) - p.lo + 8u + 15u) >> 4;  // 8 bytes of slack for the 12-byte windows
        p.off = d.head.x * 16u + p.lo;
        return p;
    };

    // requests the wavefront's half of strip i's tile
    auto request = [&](Stage& st, const Round& r, int i, const Tiles& d, const Parts& p) SD2_INLINE {
        if constexpr (FMT == kWideBitmask) {
            const uint32_t off = wide_lane(p.off, 16 * i), last = wide_lane(p.n16, 16 * i) - 1u;
#pragma unroll
            for (int c = 0; c < 2; ++c) st.v[c] = *reinterpret_cast<const u32x4*>(a.vals + (off + min((uint32_t)(c * 64 + lane), last) * 16u));
            st.tail = *reinterpret_cast<const uint2*>(a.vals + (off + min(256u + lane, 2u * last + 1u) * 8u));
            st.mk = *reinterpret_cast<const uint32_t*>(a.masks + (wide_lane(d.t, 16 * i) * 512u + 4u * my_half + (uint32_t)lane * 8u));
        } else if constexpr (FMT == kWideNm24) {
            const uint8_t* src = a.tiles + (size_t)wide_lane(d.t, 16 * i) * kNm24TileBytes;
#pragma unroll
            for (int q = 0; q < 2; ++q) st.v[q] = *reinterpret_cast<const u32x4*>(src + 1024 * (2 * my_half + q) + (uint32_t)lane * 16u);
            st.idx = *reinterpret_cast<const uint32_t*>(src + 4096 + 4 * my_half + (uint32_t)lane * 8u);
        } else {
            // columns past the matrix are cleared at the use, rows past it are not written: any element of the row will do
            const bool on = live(r, i);
            const int col0 = on ? 128 * unit_at(r) : 0, row0 = on ? strip_of(ord_at(r, i)) * 16 : 0;
            const int col = min(col0, a.k_in - 64);
            int l = lane;
            asm volatile("" : "+v"(l));  // the offsets are cheap; kept over the loop they would cost the registers of the stream
#pragma unroll
            for (int j = 0; j < 4; ++j)
                st.v[j] = block_piece(a.w + (size_t)row0 * a.k_in + col, 4 * j, min(15, a.n_out - 1 - row0), a.k_in - col, a.k_in, l);
        }
    };

    // The unit's activations: operand B of token group tg, columns 64 q + 16 g + 8 e of the unit in b[tg][2 q + e].
    // Columns past the matrix are zero; tokens past the last repeat it (their results are not written).
    u32x4 b[TG][4];
    auto load_b = [&](int u) SD2_INLINE {  // first half: the loads
        int l = lane;
        asm volatile("" : "+v"(l));
        const int col0 = min(128 * u, a.k_in - 64);
#pragma unroll
        for (int tg = 0; tg < TG; ++tg)
#pragma unroll
            for (int j = 0; j < 4; ++j) b[tg][j] = block_piece(a.x + col0, 16 * tg + 4 * j, a.k_tok - 1, a.k_in - col0, a.k_in, l);
    };
    auto turn_b = [&](int u) SD2_INLINE {  // second half, once they have landed
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) {
            asm volatile("" : "+v"(b[tg][0]), "+v"(b[tg][1]), "+v"(b[tg][2]), "+v"(b[tg][3]));
            block_to_operands(b[tg], buf, lane);
            const int col = 128 * u + 16 * g;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (col + 64 * (j >> 1) >= a.k_in) b[tg][j] = u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto op = [&](const u32x4& q) SD2_INLINE { return __builtin_bit_cast(bf16x8, q); };

    f32x4 acc[SG][TG];
    auto clear = [&]() SD2_INLINE {
#pragma unroll
        for (int i = 0; i < SG; ++i)
#pragma unroll
            for (int tg = 0; tg < TG; ++tg) acc[i][tg] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto barrier = [&]() SD2_INLINE {  // orders LDS only: loads stay in flight
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // The strips of a group are complete: strip o of the group, wavefront kw of the contraction, token group tg has its block in
    // red[((o wk + kw) TG + tg) 256 ..]; the threads share the adding, four rows of a token each.
    auto finish = [&](int grp) SD2_INLINE {
        if (!kApart) barrier();  // the slots take the place of the buffers, which some wavefront may still be reading
#pragma unroll
        for (int i = 0; i < SG; ++i)
#pragma unroll
            for (int tg = 0; tg < TG; ++tg)
                *reinterpret_cast<f32x4*>(red + ((size_t)((sw * SG + i) * wk + kw) * TG + tg) * 256 + lane * 4) = acc[i][tg];
        barrier();
        const int n_here = min(group, my_strips - grp * group);
        auto sum = [&](int o, int tg) SD2_INLINE {
            const float* p = red + ((size_t)o * wk * TG + tg) * 256 + lane * 4;
            f32x4 v = *reinterpret_cast<const f32x4*>(p) + *reinterpret_cast<const f32x4*>(p + TG * 256);
            if (W == 8 && wk == W) {  // all reads in flight at once (twelve would not leave the loop its registers)
                f32x4 q[W];
#pragma unroll
                for (int k = 2; k < W; ++k) q[k] = *reinterpret_cast<const f32x4*>(p + k * (TG * 256));
#pragma unroll
                for (int k = 2; k < W; ++k) v += q[k];
                return v;
            }
            for (int k = 2; k < wk; k += 2) {
                v += *reinterpret_cast<const f32x4*>(p + (size_t)k * (TG * 256));
                v += *reinterpret_cast<const f32x4*>(p + (size_t)(k + 1) * (TG * 256));
            }
            return v;
        };
        for (int item = wave; item < (gated ? n_here / 2 : n_here) * TG; item += W) {
            const int o = item / TG, tg = item - o * TG, tok = 16 * tg + n;
            const int ord = grp * group + o;
            if (gated) {
                const f32x4 gv = sum(2 * o, tg), uv = sum(2 * o + 1, tg);
                if (tok < a.k_tok) {
                    float m[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) m[e] = gv[e] / (1.0f + expf(-gv[e])) * uv[e];
                    const int row = strip_of(2 * o + grp * group) * 16 + 4 * g;
                    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.out) + (size_t)tok * (a.n_out / 2) + row) =
                        make_uint2(pack_bf16(m[0], m[1]), pack_bf16(m[2], m[3]));
                }
            } else {
                const f32x4 v = sum(o, tg);
                const int row = (s0 + ord) * 16 + 4 * g;
                if (tok < a.k_tok) {
                    float* dst = a.out + ((size_t)split * a.k_tok + tok) * a.n_out + row;
                    if ((a.n_out & 3) == 0) {
                        if (row < a.n_out) *reinterpret_cast<f32x4*>(dst) = v;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (row + e < a.n_out) dst[e] = v[e];
                    }
                }
            }
        }
        if (grp + 1 < n_grp) barrier();  // the slots are free again
    };

    Stage st[SG];  // each is requested for the next round as soon as it is used: a round's worth is in flight
    Round cur{0, 0}, ahead = next(cur);
    Tiles tl = directory(cur), tl_next = directory(ahead);
    // the first unit's activations go out in front of the stream: behind it they would wait for all of it
    int have_b = unit_at(cur);
    load_b(have_b);
    Parts parts = parts_of(tl);
#pragma unroll
    for (int i = 0; i < SG; ++i) request(st[i], cur, i, tl, parts);
    turn_b(have_b);
    clear();
    const uint32_t lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)reinterpret_cast<const uint8_t*>(buf);
    // LDS byte addresses of a round's runs, and which of its halves do not fit the staged part
    uint32_t runs = 0u, dense = 0u;
    auto set_runs = [&](const Tiles& d, const Parts& p) SD2_INLINE {
        if (FMT != kWideBitmask) return;
        runs = lds + d.run * 2u - p.lo;
        const unsigned long long over = __ballot(p.n16 * 16u > kWideStaged);
        dense = (uint32_t)(over & 1u) | ((uint32_t)(over >> 15) & 2u) | ((uint32_t)(over >> 30) & 4u) | ((uint32_t)(over >> 45) & 8u);
    };
    set_runs(tl, parts);
#pragma unroll 1
    for (int r = 0; r < n_rounds; ++r) {
        const Round after = next(ahead);
        const Parts parts_next = parts_of(tl_next);
        const Tiles tl_after = directory(after);
        const int u = unit_at(cur);
        const bool unit_on = u < a.n_units;
        // (a plain select becomes a branch with copies of the masks, which wait for their loads)
        const uint32_t keep = (uint32_t)__builtin_amdgcn_readfirstlane(unit_on ? -1 : 0);
        // dense: the absent half of the last unit is cleared (infinity times zero is not zero)
        const uint32_t whole = (uint32_t)__builtin_amdgcn_readfirstlane(128 * u + 128 > a.k_in ? 0 : -1);
        if (u != have_b) {
            have_b = u;
            load_b(u);
            // waited for here: a wait at the use, on every strip, would take the requests in flight with it
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            turn_b(u);
        }
        // bitmask: the step whose reads are in flight and the one being used (one where the registers do not hold two)
        WideWindow win[2];
        auto use = [&](int k) SD2_INLINE {  // step k of the round: strip k / 2, step k % 2 of its half
            Frag f0, f1;
            wide_fragments(win[kAhead ? k & 1 : 0], f0, f1);
            const int i = k >> 1, q = k & 1;
#pragma unroll
            for (int tg = 0; tg < TG; ++tg)
                acc[i][tg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f0.v, op(b[tg][2 * q]), acc[i][tg], 0, 0, 0);
#pragma unroll
            for (int tg = 0; tg < TG; ++tg)
                acc[i][tg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f1.v, op(b[tg][2 * q + 1]), acc[i][tg], 0, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < SG; ++i) {
            Stage& s = st[i];
            if constexpr (FMT == kWideBitmask) {
                reinterpret_cast<u32x4*>(buf)[lane] = s.v[0];
                reinterpret_cast<u32x4*>(buf)[64 + lane] = s.v[1];
                reinterpret_cast<uint2*>(buf)[256 + lane] = s.tail;
                if (dense >> i & 1u) {  // the rest of a dense half's stream is fetched here
                    const u32x4* s16 = reinterpret_cast<const u32x4*>(a.vals + wide_lane(parts.off, 16 * i));
                    const uint32_t n16 = wide_lane(parts.n16, 16 * i);
                    for (uint32_t c = kWideStaged / 16 + lane; c < n16; c += 64) reinterpret_cast<u32x4*>(buf)[c] = s16[c];
                }
                const uint32_t mk = s.mk & keep;
                request(s, ahead, i, tl_next, parts_next);
                asm volatile("" ::: "memory");  // the request goes out before the expansion, not after it
                uint32_t ex[2];
                wide_scan(mk, ex);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int k = 2 * i + q;
                    wide_reads(win[kAhead ? k & 1 : 0], runs, 16 * i + 4 * q, lut, ex[q], q ? mk >> 16 : mk);
                    asm volatile("" ::: "memory");
                    if (!kAhead)
                        use(k);
                    else if (k > 0)
                        use(k - 1);
                }
            } else if constexpr (FMT == kWideNm24) {
                if (unit_on) {
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int tg = 0; tg < TG; ++tg) {
                            Frag16 bq;
                            bq.q[0] = b[tg][2 * q];
                            bq.q[1] = b[tg][2 * q + 1];
                            acc[i][tg] = q ? __builtin_amdgcn_smfmac_f32_16x16x64_bf16(op(s.v[q]), bq.v, acc[i][tg], (int)s.idx, 0, 1)
                                           : __builtin_amdgcn_smfmac_f32_16x16x64_bf16(op(s.v[q]), bq.v, acc[i][tg], (int)s.idx, 0, 0);
                        }
                }
                request(s, ahead, i, tl_next, parts_next);
            } else {
                u32x4 w[4] = {s.v[0], s.v[1], s.v[2], s.v[3]};
                block_to_operands(w, buf, lane);
                w[2] &= whole;
                w[3] &= whole;
                request(s, ahead, i, tl_next, parts_next);
                asm volatile("" ::: "memory");
                if (unit_on) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int tg = 0; tg < TG; ++tg) acc[i][tg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op(w[j]), op(b[tg][j]), acc[i][tg], 0, 0, 0);
                }
            }
        }
        if (FMT == kWideBitmask && kAhead) use(2 * SG - 1);
        if (cur.pass + 1 == n_pass) {
            finish(cur.grp);
            clear();
        }
        cur = ahead;
        ahead = after;
        set_runs(tl_next, parts_next);
        parts = parts_next;
        tl_next = tl_after;
    }
}

// ---------------------------------------------------------------- plan and launch

// How a wide linear is cut.  The model behind the choice is a fit to this part, in microseconds: a strip costs a pass the
// expansion of its half tile (two or three wavefronts on a SIMD take turns), fetching a unit's activations is paid once a
// pass and grows with the tokens, completing a group takes 1.5, and a partial result its bytes to memory and back plus a
// launch where nothing adds it anyway, and where the norm does, from nine on, 1.5 for a second trip of its loads (1.5B shape on 64
// tokens, down: five partial results and two passes in place of nine and one, a layer 67.8 -> 66.5 us).  Twelve wavefronts where
// their 168 registers hold the sums of a group.
bool wide_plan(int n_out, int k_in, int n_strips, int k_tok, bool gated, int max_split, bool free_add, WidePlan* out) {
    const int tg = (k_tok + 15) / 16;
    if (tg < 2 || tg > 4 || (gated && n_out % 32) || k_in > (1 << 20) || (int64_t)n_out * k_in > (1ll << 31) - (1 << 23))
        return false;  // 32-bit byte offsets, into the value section and over 64 rows of activations
    const int n_units = (k_in + 127) / 128;
    const int cus = device_cu_count(), step = gated ? 2 : 1;
    const int max_cut = std::min(std::min(max_split, kWideMaxSplit), std::min(n_units, cus));
    int per_wg[kWideMaxSplit + 1], units[kWideMaxSplit + 1];  // strips of a workgroup, units of a split
    double extra[kWideMaxSplit + 1];
    for (int split = 1; split <= max_cut; ++split) {
        const int blocks = std::max(1, std::min(n_strips / step, cus / split));
        per_wg[split] = step * ((n_strips / step + blocks - 1) / blocks);
        units[split] = (n_units + split - 1) / split;
        extra[split] = split > 1 ? (double)split * k_tok * n_out * 8.0 / 4e6 + (!free_add ? 3.0 : split > 8 ? 1.5 : 0.0) : 0.0;
    }
    double best = -1.0;
    for (int waves = 8; waves <= 12; waves += 4)
        for (int sg = 2; sg <= 4; ++sg) {
            if (waves == 12 && tg * sg > 6) continue;
            const double pass = waves == 8 ? sg * (0.7 + 0.06 * tg) + 0.3 + 0.45 * tg : sg * (0.95 + 0.06 * tg) + 0.3 + 0.6 * tg;
            for (int wk = waves; wk >= 2; wk -= 2) {
                if (waves % wk) continue;
                const int group = sg * (waves / wk);
                if (gated && group % 2) continue;  // pairs stay within a group
                for (int split = 1; split <= max_cut; ++split) {
                    const int n_pass = (units[split] + wk - 1) / wk;
                    if ((split - 1) * n_pass * wk >= n_units) continue;  // an empty split
                    const int groups = (per_wg[split] + group - 1) / group;
                    const double t = groups * (n_pass * pass + 1.5) + extra[split];
                    if (best < 0.0 || t < best) {
                        best = t;
                        out->waves = waves;
                        out->n_split = split;
                        out->n_pass = n_pass;
                        out->wk = wk;
                        out->sg = sg;
                    }
                }
            }
        }
    if (best >= 0.0) {
        out->strips_per_wg = per_wg[out->n_split];
        out->n_wg = out->n_split * ((n_strips + out->strips_per_wg - 1) / out->strips_per_wg);
        out->n_units = n_units;
    }
    return best >= 0.0;
}

template <int FMT, int TG, int SG, int W>
static hipError_t launch_wide_t(const WideArgs& a, const WidePlan& p, hipStream_t s) {
    constexpr size_t buffers = (size_t)W * kWideBufDw * 4, sums = wide_sums_bytes(SG, TG, W);
    constexpr size_t lds = wide_apart(SG, TG, W) ? buffers + sums : std::max(buffers, sums);
    static std::atomic<bool> raised{false};
    if (!raised.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wide_linear_kernel<FMT, TG, SG, W>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        raised.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((wide_linear_kernel<FMT, TG, SG, W>), dim3((unsigned)p.n_wg), dim3(64 * W), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_wide_linear(const MatArgs& m, bool nm24, const uint16_t* x, int k_tok, void* out, bool gated, const WidePlan& p,
                              hipStream_t s) {
    WideArgs a;
    a.dir = static_cast<const uint8_t*>(m.dir);
    a.masks = reinterpret_cast<const uint8_t*>(m.masks);
    a.vals = reinterpret_cast<const uint8_t*>(m.vals);
    a.tiles = static_cast<const uint8_t*>(m.dir);
    a.w = m.w;
    a.x = x;
    a.out = static_cast<float*>(out);
    a.n_out = m.n_out;
    a.k_in = m.k_in;
    a.k_tok = k_tok;
    a.n_strips = m.n_strips;
    a.n_units = p.n_units;
    a.n_split = p.n_split;
    a.n_pass = p.n_pass;
    a.wk = p.wk;
    a.strips_per_wg = p.strips_per_wg;
    a.half_strips = gated ? m.n_strips / 2 : 0;
    if (gated && p.n_split != 1) return hipErrorInvalidValue;
    const int fmt = m.w ? kWideDense : (nm24 ? kWideNm24 : kWideBitmask), tg = (k_tok + 15) / 16;
#define SD2_WIDE_SG(F, T, S) \
    if (p.sg == S && p.waves == 8) return launch_wide_t<F, T, S, 8>(a, p, s); \
    if constexpr (T * S <= 6) \
        if (p.sg == S && p.waves == 12) return launch_wide_t<F, T, S, 12>(a, p, s)
#define SD2_WIDE_CASE(F, T) \
    if (fmt == F && tg == T) { \
        SD2_WIDE_SG(F, T, 2); \
        SD2_WIDE_SG(F, T, 3); \
        SD2_WIDE_SG(F, T, 4); \
        return hipErrorInvalidValue; \
    }
    SD2_WIDE_CASE(kWideBitmask, 2)
    SD2_WIDE_CASE(kWideBitmask, 3)
    SD2_WIDE_CASE(kWideBitmask, 4)
    SD2_WIDE_CASE(kWideNm24, 2)
    SD2_WIDE_CASE(kWideNm24, 3)
    SD2_WIDE_CASE(kWideNm24, 4)
    SD2_WIDE_CASE(kWideDense, 2)
    SD2_WIDE_CASE(kWideDense, 3)
    SD2_WIDE_CASE(kWideDense, 4)
#undef SD2_WIDE_CASE
#undef SD2_WIDE_SG
    return hipErrorInvalidValue;
}

}  // namespace sd2
