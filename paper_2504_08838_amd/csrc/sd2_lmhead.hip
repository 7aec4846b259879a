// libsd2 -- the drafter's LM head with the greedy choice fused in (gfx950).
//
// Eq. 1 (Sec. 2.1) draws each draft token from the drafter's distribution; greedy drafting takes
// the largest logit.  The head is the one linear that is never pruned (Sec. 2.3, Sec. 3.2), so it
// is a plain dense [vocab][hidden] bf16 matrix streamed once per call: pure HBM traffic.
//
// One workgroup of 8 wavefronts per compute unit walks over 16-row strips of the matrix.  Inside a
// workgroup the contraction is split eight ways: wavefront w owns the 128-column chunks w, w+8, ...
// of every strip, and keeps the matching slice of the normalised activations (operand B of the
// MFMAs) in registers for the whole kernel.  Weights travel HBM -> LDS directly
// (16-byte buffer requests, 256 contiguous bytes per row piece) into a per-wave ring of four 4 KiB
// chunk buffers, refilled as soon as its reads have returned, so up to four chunks are in flight; the 16-byte
// pieces of a row are stored xor-swizzled by the row number so that the MFMA-layout reads
// (one row per lane) hit sixteen different bank groups.  Per strip the eight partial 16 x 16
// results meet in LDS (double buffered, one barrier), four wavefronts add them in a fixed order and
// keep a running (largest logit, lowest row) per thread; nothing but 16 candidates per workgroup
// ever goes back to HBM unless the caller asks for the logits.
#include <algorithm>
#include <atomic>

#include "sd2_device.h"
#include "sd2_internal.h"

namespace sd2 {

constexpr int kLmWaves = 8;                     // wavefronts per workgroup = ways the contraction is split
constexpr int kLmChunkCols = 128;               // columns of one staged chunk (16 rows x 128 x bf16 = 4 KiB)
constexpr int kLmRing = 4;                      // chunk buffers per wavefront
constexpr int kLmChunkDw = 16 * kLmChunkCols / 2;
constexpr int kLmRedDw = kLmWaves * 256;        // one set of partial strips
constexpr int kLmMiscDw = kLmWaves * 16 + 512;  // sums of squares per block of columns and token; final candidates (behind the first 128)
constexpr int kLmNowhereDw = 256;                // where requests for nothing lead; nobody reads it
constexpr int kLmThirdDw = kLmWaves / 2 * 512;   // squares of a third block of columns on their way between neighbours
constexpr int kLmLdsDw = kLmWaves * kLmRing * kLmChunkDw + 2 * kLmRedDw + kLmMiscDw + kLmThirdDw + kLmNowhereDw;
static_assert(kLmLdsDw * 4 <= 160 * 1024, "a workgroup fits a compute unit");

struct LmCand {
    float v;
    int32_t i;
};

// (a, ia) <- the better of the two: larger value, on equal values the lower index
__device__ __forceinline__ void lm_better(float& a, int32_t& ia, float b, int32_t ib) {
    if (b > a || (b == a && ib < ia)) {
        a = b;
        ia = ib;
    }
}

// What a launch of the kernel is.  kHead: the LM head (fp32 residual in `h`, final norm, greedy choice, logits optional).  The others
// are the same stream as a dense linear, y = x W^T with every sum final inside the workgroup:
//   kPlain  every result written to `out` ([k_tok][vocab] with vocab = n_out)
//   kGated  the matrix is [gate; up]: a strip is eight rows of each half, and bf16(silu(gate) * up) leaves as the next linear's
//           activations ([k_tok][vocab / 2] bf16 in `out`): no launch for the product and no fp32 results in memory.  Eight rows
//           and eight, not pairs of strips: as many strips as the plain linear has, so the workgroups share them as evenly.
//   kAdd    results are added to the residual stream `out`; a workgroup has one strip (n_out <= 4096), whose residual is requested first
// NORM: the activations are the RMS norm of the fp32 residual `h` (in place of bf16 `x`).  Every workgroup normalises for itself:
// it reads twice the bytes of `x` from L2, and a launch with its gap (about 4 us) goes.
// Dense stacks of 8 layers, us, every step a launch of its own and the activations behind the stream, then now: hidden 3072 on 5 tokens
// 498 -> 436, on 16 tokens 574 -> 519; hidden 4096 on 5 tokens 612 -> 572; MLP 2048 x 8192 on 5 tokens 28.1 -> 24.2.
//   kAtt    as kAdd, and the activations are the context of the attention among the in-flight tokens: column chunk c is head c, so a
//           wavefront attends for the heads whose columns it multiplies, from q|k|v in `h`, and a launch goes.  Made for 2 or 5 token
//           slots; with more scores than that a launch of its own is faster (dense_stream_attend_ok).
enum { kLmHead, kLmPlain, kLmGated, kLmAdd, kLmAtt2, kLmAtt5 };
constexpr int lm_att_slots(int mode) { return mode == kLmAtt2 ? 2 : mode == kLmAtt5 ? 5 : 0; }

// HALF: a strip is eight rows (kPlain, kAdd and kAtt with one strip a workgroup and one pass): a chunk is two requests instead of four,
// the matrix instructions' other eight rows are whatever the ring holds and nobody reads their results.  Twice the compute units stream.
// A row's columns, wavefronts and order of sums are those of sixteen rows.
// As a linear TG = 2 takes up to 32 tokens in one pass (two sets of B operands in registers, two accumulators per strip; the partial
// strips then share one LDS buffer and need a second barrier per strip).
template <int CPW, int MODE, bool NORM, int TG, bool HALF>
__global__ __launch_bounds__(64 * kLmWaves) void lm_head_kernel(const uint16_t* __restrict__ w,
                                                                const float* __restrict__ h,
                                                                const uint16_t* __restrict__ x_all, int vocab, int hidden,
                                                                int k_tok_all, int rep, LmCand* __restrict__ part,
                                                                float* __restrict__ out_all) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lm_smem[];
    constexpr bool HEAD = MODE == kLmHead, ADD = MODE >= kLmAdd;
    constexpr int kSlots = lm_att_slots(MODE);
    constexpr int kLoads = HALF ? 2 : 4, kRows = MODE == kLmGated || HALF ? 8 : 16;  // requests of a chunk; rows of a strip (of each half)
    static_assert(!HALF || (MODE != kLmHead && MODE != kLmGated && TG == 1), "eight rows a strip as a linear");
    // As a linear with more tokens than one pass takes, the grid's second dimension numbers the passes of 16 TG
    // tokens (the matrix is streamed once per pass); the head itself is launched with one pass.
    const int pass = HEAD ? 0 : (int)blockIdx.y;
    const int n_cols_out = MODE == kLmGated ? vocab / 2 : vocab;
    const uint16_t* __restrict__ x = (HEAD || NORM || kSlots) ? x_all : x_all + (size_t)pass * (16 * TG) * hidden;
    float* __restrict__ logits = (HEAD || MODE == kLmGated) ? out_all : out_all + (size_t)pass * (16 * TG) * vocab;
    uint16_t* __restrict__ gated = reinterpret_cast<uint16_t*>(out_all) + (size_t)pass * (16 * TG) * n_cols_out;
    const int k_tok = HEAD ? k_tok_all : min(16 * TG, k_tok_all - pass * (16 * TG));
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    uint32_t* ring = lm_smem + wave * (kLmRing * kLmChunkDw);
    float* red = reinterpret_cast<float*>(lm_smem + kLmWaves * kLmRing * kLmChunkDw);
    float* misc = red + 2 * kLmRedDw;

    // Made here and not an argument: with one more, the grid's size lies in a second cache line of the arguments, and every launch waits
    // for that line's trip, too (0.2 us; dense stacks of four layers, hidden 3072 on 12 tokens 252.5 -> 249.1, hidden 1536 on 5 141.7 -> 139.6).
    const int n_strips = HALF ? (vocab + 7) / 8 : (vocab + 15) / 16;
    const int n_colchunks = hidden / kLmChunkCols;
    const int my_strips = (n_strips - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    constexpr int kSure = CPW == 6 || CPW == 8 ? CPW - 2 : CPW - 1;  // column chunks that every wavefront has (6 and 8 also serve 5 and 7)
    int n_cc = 0;                                                    // this wavefront's: wave + 8 cc
#pragma unroll
    for (int cc = 0; cc < CPW; ++cc) n_cc += wave + kLmWaves * cc < n_colchunks ? 1 : 0;
    const int n_chunks = my_strips * n_cc;

    static_assert(kLmRing == 4, "the waits below count three chunks behind the current one");
    // The wavefront's chunks, in order: its n_cc column chunks of strip blockIdx.x, then of strip blockIdx.x + gridDim.x, ...
    // Instruction i of a chunk fills LDS rows 4i..4i+3 (16 lanes per row); lane l brings the 16-byte piece
    // (l & 15) ^ row of its row, so piece j of row r sits at LDS piece position j ^ r.
    // Requested as a buffer that starts at the chunk and ends with its last row: only its base is per request, in scalars, and
    // rows past the matrix ask memory for nothing (the hardware's range check).  It also lets the compiler count these requests where
    // it waits for the activations; global-memory requests into LDS make it wait for all.  What does not exist is not requested
    // either: a request that the range check empties costs as much issue as a full one (three of them per wavefront
    // at the end cost a linear 0.7 us).
    uint32_t piece[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 4 * i + g;
        piece[i] = (uint32_t)((MODE == kLmGated ? 4 * (i & 1) + g : r) * hidden + ((n ^ r) * 8)) * 2u;
    }
    int issued = 0, r_strip = 0, r_cc = 0;  // chunks requested; the next one's strip and column chunk
    auto request_chunk = [&](bool exists) {
        // a request for nothing must not lead to the slot that the next chunk takes while it is in flight
        uint32_t* dst = exists ? ring + (issued & (kLmRing - 1)) * kLmChunkDw : lm_smem + kLmLdsDw - kLmNowhereDw;
        const int step = exists ? 256 : 0;
        const int row = ((int)blockIdx.x + r_strip * (int)gridDim.x) * kRows;
        const int rows = MODE == kLmGated ? 8 : min(kRows, vocab - row);
        const int bytes = exists ? ((rows - 1) * hidden + kLmChunkCols) * 2 : 0;
        const uint16_t* src = w + (size_t)row * hidden + (wave + kLmWaves * r_cc) * kLmChunkCols;
        const auto rows_lo = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(src), 0, bytes, 0x00020000);
        const auto rows_hi = MODE == kLmGated
                                 ? __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(src + (size_t)n_cols_out * hidden), 0, bytes, 0x00020000)
                                 : rows_lo;
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(i < 2 ? rows_lo : rows_hi, (__attribute__((address_space(3))) void*)(dst + i * step), 16,
                                                     (int)piece[i], 0, 0, 0);
        issued += exists ? 1 : 0;
        r_cc += exists ? 1 : 0;
        if (r_cc >= n_cc) {
            r_cc = 0;
            ++r_strip;
        }
    };
    auto issue_chunk = [&]() {
        if (issued < n_chunks) request_chunk(true);
    };
    // Chunk ci has landed once at most the loads of the chunks issued after it are outstanding (loads return in
    // order): up to three chunks of kLoads loads each, fewer at the end of the wavefront's work.
    auto wait_chunk = [&](int ci) {
        const int later = min(n_chunks - 1 - ci, kLmRing - 1);
        if (later >= 3)
            __builtin_amdgcn_s_waitcnt(0x0F70 | (3 * kLoads));
        else if (later == 2)
            __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * kLoads));
        else if (later == 1)
            __builtin_amdgcn_s_waitcnt(0x0F70 | kLoads);
        else
            __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("" ::: "memory");
    };

    static_assert(TG == 1 || (!HEAD && !NORM), "the norm takes one token group per pass");
    static_assert(!NORM || CPW <= 4, "the residual's columns of a wavefront fit its registers");
    const int tok = min(n, k_tok - 1);  // lanes past the last token repeat it; their results are never used
    // Reducing thread (wave rho < 4, lane l) owns result element l of source lane group rho: token l >> 2,
    // row 4 rho + (l & 3) of each strip, so its running best needs no cross-lane work until the very end.
    const int red_tok = lane >> 2, red_row = 4 * wave + (lane & 3);
    float residual = 0.f;
    Frag b[TG][CPW][4];
    if (HEAD && !NORM) {
#pragma unroll
        for (int c = 0; c < kLmRing; ++c) issue_chunk();
        // ---- final norm of the residual stream, straight into operand B: a = bf16(h / sqrt(mean(h^2) + eps))
        for (int t = 0; t < k_tok; ++t) {
            float s = 0.f;
            for (int c = tid * 4; c < hidden; c += 64 * kLmWaves * 4) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(h + (size_t)t * hidden + c);
                s += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
            if (lane == 0) misc[wave * 16 + t] = s;
        }
        __syncthreads();
        float tot = 0.f;
#pragma unroll
        for (int ww = 0; ww < kLmWaves; ++ww) tot += misc[ww * 16 + tok];
        const float inv = 1.0f / sqrtf(tot / (float)hidden + 1e-5f);
#pragma unroll
        for (int cc = 0; cc < CPW; ++cc) {
            const int colchunk = wave + kLmWaves * cc;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (colchunk < n_colchunks) {
                    const float* src = h + (size_t)tok * hidden + colchunk * kLmChunkCols + (q * 4 + g) * 8;
                    const f32x4 lo = *reinterpret_cast<const f32x4*>(src);
                    const f32x4 hi = *reinterpret_cast<const f32x4*>(src + 4);
                    b[0][cc][q].u[0] = pack_bf16(lo[0] * inv, lo[1] * inv);
                    b[0][cc][q].u[1] = pack_bf16(lo[2] * inv, lo[3] * inv);
                    b[0][cc][q].u[2] = pack_bf16(hi[0] * inv, hi[1] * inv);
                    b[0][cc][q].u[3] = pack_bf16(hi[2] * inv, hi[3] * inv);
                } else {
                    b[0][cc][q].q = u32x4{0u, 0u, 0u, 0u};  // column chunk past the matrix: contributes nothing
                }
            }
        }
    } else {
        // The activations are requested in front of the wavefront's stream and without branches, so that their wait leaves the stream
        // in flight.  Behind it they came with its last byte (loads return in the order of their issue): the ring was full and
        // idle until then, and nothing was requested meanwhile.  A barrier that puts every wavefront's in front of anybody's stream
        // costs more than it gives here: 55 us a layer against 52.5 (hidden 3072, 5 tokens), the stream starts later.
        f32x4 hr[NORM ? CPW : 1][4][2];
        FewTokens<kSlots ? kSlots : 1> heads[kSlots ? CPW : 1];
        if (ADD) {
            const int row = (int)blockIdx.x * kRows + red_row;
            if (wave < kRows / 4 && row < vocab && red_tok < k_tok) residual = logits[(size_t)red_tok * vocab + row];
        }
        if constexpr (kSlots > 0) {
            const int kv_out = n_colchunks / rep * kLmChunkCols;
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
                const int head = min(wave + kLmWaves * cc, n_colchunks - 1), at = hidden + head / rep * kLmChunkCols;
                load_few(heads[cc], h, hidden + 2 * kv_out, head * kLmChunkCols, at, at + kv_out, k_tok, lane);
            }
        }
#pragma unroll
        for (int cc = 0; cc < (kSlots ? 0 : CPW); ++cc) {
            const size_t col = (size_t)min(wave + kLmWaves * cc, n_colchunks - 1) * kLmChunkCols + g * 8;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (NORM) {
                    const float* src = h + (size_t)tok * hidden + col + q * 32;
                    hr[cc][q][0] = *reinterpret_cast<const f32x4*>(src);
                    hr[cc][q][1] = *reinterpret_cast<const f32x4*>(src + 4);
                } else {
#pragma unroll
                    for (int tg = 0; tg < TG; ++tg)
                        b[tg][cc][q].q = *reinterpret_cast<const u32x4*>(x + (size_t)min(n + 16 * tg, k_tok - 1) * hidden + col + q * 32);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // all of them on their way before the first is waited for
#pragma unroll
        for (int c = 0; c < CPW && c < kLmRing; ++c) request_chunk(c < kSure || c < n_cc);  // the first strip's: without a branch
        __builtin_amdgcn_sched_barrier(0);
        // The rest of the ring, once the activations are there.  (Behind the whole norm, dense stack of 28 layers, hidden 1536, 5 tokens: 1131 us
        // against 1106.)
        auto fill_ring = [&]() {
#pragma unroll
            for (int c = 0; c < kLmRing; ++c)
                if (issued < kLmRing) issue_chunk();
        };
        if (NORM) {
            // The sum of squares, in the order in which a launch of its own adds it (residual_norm_kernel; for the head, the prologue
            // above), so that the same residual gives the same activations on either way.  That order: four columns, then a tree over the
            // 64 such groups of 256 columns whose first step adds columns 128 apart, then the blocks of 256 columns in turn.  Here
            // lane (n, g) of wavefront w has token n's groups (q, e) = columns 32 q + 8 g + 4 e of its column chunks, and the columns
            // 128 away are the neighbouring wavefront's.  Neighbours meet in the room of the partial strips, two chunks at a time (three
            // chunks at once, by way of room of its own for the third): of the first chunk's block the even wavefront adds up all, of the
            // second's the odd one, of the third's the even one again.  (Adding in whatever order was nearest cost
            // 0.4 us less a launch and moved a dense stack's outputs by 2e-3: other bf16 neighbours.)
            constexpr int kBlocks = HEAD && CPW > 2 ? 2 : CPW;  // the head's threads first add their columns 2048 apart
            constexpr int kTokDw = 4 * kBlocks + 4;             // a token's blocks, and a piece to spread the tokens over the banks
            static_assert(!NORM || (16 * kTokDw <= kLmMiscDw && kLmRedDw % 4 == 0), "the blocks' sums fit, 16-byte aligned");
            const bool odd = wave & 1;
            auto squares = [&](int cc, f32x4 (&sq)[2]) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        sq[e][q] = 0.f;
#pragma unroll
                        for (int c = cc; c < CPW; c += kBlocks) {
                            const f32x4 v = hr[c][q][e];
                            const float s = HEAD ? v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]
                                                 : (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
                            sq[e][q] += wave + kLmWaves * c < n_colchunks ? s : 0.f;
                        }
                    }
            };
            auto meet = [&]() {
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            };
            // adds up a block whose squares are in `v` and, of the neighbour, at `get`
            auto add_up = [&](const f32x4 (&v)[2], const f32x4* get, int block) {
                float s[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const f32x4 both = v[e] + get[64 * e];
                    s[e] = (both[0] + both[2]) + (both[1] + both[3]);
                }
#pragma unroll
                for (int o = 32; o >= 16; o >>= 1)
#pragma unroll
                    for (int e = 0; e < 2; ++e) s[e] += __shfl_xor(s[e], o);
                if (lane < 16) misc[lane * kTokDw + (wave >> 1) + 4 * block] = s[0] + s[1];
            };
            constexpr bool kThird = kBlocks == 3;
            f32x4* third_at = reinterpret_cast<f32x4*>(misc + kLmMiscDw) + (wave >> 1) * 128 + lane;
#pragma unroll
            for (int c0 = 0; c0 < (kThird ? 1 : kBlocks); c0 += 2) {
                // the second pair of chunks goes where this wavefront has just read of the first (nobody else reads there)
                f32x4* put = reinterpret_cast<f32x4*>(red) + (c0 ? wave : wave ^ 1) * 128 + lane;
                const f32x4* get = reinterpret_cast<const f32x4*>(red) + (c0 ? wave ^ 1 : wave) * 128 + lane;
                const bool pair = c0 + 1 < kBlocks;
                f32x4 first[2], second[2], third[2], v[2];
                squares(c0, first);
                squares(pair ? c0 + 1 : c0, second);
                if (kThird) squares(kBlocks - 1, third);
                if (odd) {
                    put[0] = first[0];
                    put[64] = first[1];
                    if (kThird) {
                        third_at[0] = third[0];
                        third_at[64] = third[1];
                    }
                    v[0] = second[0];
                    v[1] = second[1];
                } else {
                    if (pair) {
                        put[0] = second[0];
                        put[64] = second[1];
                    }
                    v[0] = first[0];
                    v[1] = first[1];
                }
                if (kThird || c0 + 2 >= kBlocks) fill_ring();  // all of the residual is there
                meet();
                if (!odd || pair) add_up(v, get, odd ? c0 + 1 : c0);
                if (kThird && !odd) add_up(third, third_at, kBlocks - 1);
                asm volatile("" ::: "memory");  // (the reads have returned: their sums are on their way)
            }
            meet();
            f32x4 blocks[kBlocks];
#pragma unroll
            for (int j = 0; j < kBlocks; ++j) blocks[j] = *reinterpret_cast<const f32x4*>(misc + n * kTokDw + 4 * j);
            float tot = 0.f;
#pragma unroll
            for (int j = 0; j < kBlocks; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) tot += blocks[j][i];
            const float inv = 1.0f / sqrtf(tot / (float)hidden + 1e-5f);
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const f32x4 v = hr[cc][q][e];
                        b[0][cc][q].u[2 * e] = pack_bf16(v[0] * inv, v[1] * inv);
                        b[0][cc][q].u[2 * e + 1] = pack_bf16(v[2] * inv, v[3] * inv);
                    }
        }
        if constexpr (kSlots > 0) {
            // The context goes from two dimensions a lane to operand B through the wavefront's own places in the two buffers of partial
            // strips (tokens 0-3, 4-7): where it leaves its strips later, and nobody else does.
            uint32_t* turn = reinterpret_cast<uint32_t*>(red) + wave * 256;
            auto place = [&](int t) { return turn + (t >> 2) * kLmRedDw + (t & 3) * 64; };
            static_assert(kSlots <= 8, "two buffers of four tokens");
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
                attend_few(heads[cc], [&](int t, float x0, float x1) { place(t)[lane] = pack_bf16(x0, x1); });
                asm volatile("" ::: "memory");
#pragma unroll
                for (int q = 0; q < 4; ++q) b[0][cc][q].q = *reinterpret_cast<const u32x4*>(place(tok) + q * 16 + g * 4);
                asm volatile("" ::: "memory");
            }
        }
        // waited for here, where what is behind them is known: in the loop the compiler would wait for the stream, too
#pragma unroll
        for (int tg = 0; tg < TG; ++tg)
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc)
                asm volatile("" : "+v"(b[tg][cc][0].q), "+v"(b[tg][cc][1].q), "+v"(b[tg][cc][2].q), "+v"(b[tg][cc][3].q));
        if (ADD) asm volatile("" : "+v"(residual));
        if (!NORM) fill_ring();
    }

    // ---- strips
    float best = -INFINITY;
    int32_t best_i = 0x7fffffff;
    int ci = 0;
#pragma unroll 1
    for (int si = 0; si < my_strips; ++si) {
        f32x4 acc[TG];
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) acc[tg] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cc = 0; cc < CPW; ++cc) {
            if (cc >= kSure && cc >= n_cc) break;
            wait_chunk(ci);
            const uint32_t* buf = ring + (ci & (kLmRing - 1)) * kLmChunkDw;
            Frag a[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q].q = *reinterpret_cast<const u32x4*>(buf + (n * 16 + ((q * 4 + g) ^ n)) * 4);
            // the buffer is refilled only after its reads have returned
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
            asm volatile("" ::: "memory");
            issue_chunk();
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int tg = 0; tg < TG; ++tg) acc[tg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[q].v, b[tg][cc][q].v, acc[tg], 0, 0, 0);
            ++ci;
        }
        // one token group: the partial strips alternate between two buffers (one barrier per strip); two groups fill
        // both buffers at once and a second barrier frees them
        float* mine = red + (TG == 1 ? (si & 1) * kLmRedDw : 0);
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) *reinterpret_cast<f32x4*>(mine + tg * kLmRedDw + wave * 256 + lane * 4) = acc[tg];
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the partial strip is in LDS; loads stay in flight
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (wave < kRows / 4) {
#pragma unroll
            for (int tg = 0; tg < TG; ++tg) {
                const int rt = red_tok + 16 * tg;
                float v = 0.f;
#pragma unroll
                for (int ww = 0; ww < kLmWaves; ++ww) v += mine[tg * kLmRedDw + ww * 256 + wave * 64 + lane];
                if (MODE == kLmGated) {  // waves 0 and 1: rows 0..7 are the gate's, rows 8..15 the same rows of up
                    float up = 0.f;
#pragma unroll
                    for (int ww = 0; ww < kLmWaves; ++ww) up += mine[tg * kLmRedDw + ww * 256 + (wave + 2) * 64 + lane];
                    if (rt < k_tok)
                        gated[(size_t)rt * n_cols_out + ((int)blockIdx.x + si * (int)gridDim.x) * 8 + red_row] = f32_to_bf16(v / (1.0f + expf(-v)) * up);
                    continue;
                }
                const int row = ((int)blockIdx.x + si * (int)gridDim.x) * kRows + red_row;
                if (row < vocab && rt < k_tok) {
                    if (HEAD && v > best) {  // rows come in increasing order: '>' keeps the lowest index among equals
                        best = v;
                        best_i = row;
                    }
                    if (!HEAD || logits) logits[(size_t)rt * vocab + row] = ADD ? residual + v : v;
                }
            }
        }
        if (TG > 1) {
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    }
    wait_vector_memory();  // nothing is on its way into LDS when the wavefront ends
    if (!HEAD) return;
    // ---- 16 threads per token hold candidates: pick one per token and workgroup
    LmCand* cand = reinterpret_cast<LmCand*>(misc + kLmWaves * 16);
    if (wave < 4) cand[wave * 64 + lane] = LmCand{best, best_i};
    __syncthreads();
    if (tid < 16) {
        float bv = -INFINITY;
        int32_t bi = 0x7fffffff;
        for (int rho = 0; rho < 4; ++rho)
            for (int j = 0; j < 4; ++j) {
                const LmCand c = cand[rho * 64 + tid * 4 + j];
                lm_better(bv, bi, c.v, c.i);
            }
        part[(size_t)blockIdx.x * 16 + tid] = LmCand{bv, bi};
    }
}

// One wavefront per token folds the candidates of all workgroups.
__global__ __launch_bounds__(1024) void lm_head_pick_kernel(const LmCand* __restrict__ part, int n_wg, int k_tok,
                                                            int32_t* __restrict__ token_ids,
                                                            float* __restrict__ max_logit) {
    const int lane = threadIdx.x & 63, t = threadIdx.x >> 6;
    if (t >= k_tok) return;
    float bv = -INFINITY;
    int32_t bi = 0x7fffffff;
    for (int j = lane; j < n_wg; j += 64) {
        const LmCand c = part[(size_t)j * 16 + t];
        lm_better(bv, bi, c.v, c.i);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o);
        const int32_t oi = __shfl_xor(bi, o);
        lm_better(bv, bi, ov, oi);
    }
    if (lane == 0) {
        token_ids[t] = bi == 0x7fffffff ? 0 : bi;  // every logit NaN: no candidate ever won
        if (max_logit) max_logit[t] = bv;
    }
}

// one per compute unit; the head's candidates have room for kLmMaxWorkgroups
static int lm_workgroups(int n_strips, bool head) {
    const int n = std::min(n_strips, device_cu_count());
    return head ? std::min(n, kLmMaxWorkgroups) : n;
}

template <int CPW, int MODE, bool NORM, int TG = 1, bool HALF = false>
static hipError_t launch_lm_t(const uint16_t* w, const float* h, const uint16_t* x, int vocab, int hidden, int k_tok, LmCand* part, float* out,
                              hipStream_t s, int rep = 1) {
    static std::atomic<bool> attr_set{false};  // more than the default 64 KiB of dynamic LDS needs opting in, once per kernel
    const size_t lds = (size_t)kLmLdsDw * 4;
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&lm_head_kernel<CPW, MODE, NORM, TG, HALF>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const int n_strips = HALF ? (vocab + 7) / 8 : (vocab + 15) / 16;
    const int n_wg = MODE >= kLmAdd ? n_strips : lm_workgroups(n_strips, MODE == kLmHead);
    const int passes = MODE == kLmHead ? 1 : (k_tok + 16 * TG - 1) / (16 * TG);
    hipLaunchKernelGGL((lm_head_kernel<CPW, MODE, NORM, TG, HALF>), dim3((unsigned)n_wg, (unsigned)passes), dim3(64 * kLmWaves), lds, s, w, h, x, vocab,
                       hidden, k_tok, rep, part, out);
    return hipGetLastError();
}

// NORM is a request: up to 4096 columns (four column chunks a wavefront) the residual's columns fit the registers
template <int MODE, bool NORM, bool HALF = false>
static hipError_t launch_lm_cpw(const uint16_t* w, const float* h, const uint16_t* x, int vocab, int hidden, int k_tok, LmCand* part, float* out,
                                hipStream_t s) {
    constexpr bool kLong = !NORM || MODE == kLmHead;  // the head has another prologue for longer rows
    switch ((hidden / kLmChunkCols + kLmWaves - 1) / kLmWaves) {
        case 1: return launch_lm_t<1, MODE, NORM, 1, HALF>(w, h, x, vocab, hidden, k_tok, part, out, s);
        case 2: return launch_lm_t<2, MODE, NORM, 1, HALF>(w, h, x, vocab, hidden, k_tok, part, out, s);
        case 3: return launch_lm_t<3, MODE, NORM, 1, HALF>(w, h, x, vocab, hidden, k_tok, part, out, s);
        case 4: return launch_lm_t<4, MODE, NORM, 1, HALF>(w, h, x, vocab, hidden, k_tok, part, out, s);
        case 5: case 6: if constexpr (kLong) return launch_lm_t<6, MODE, false, 1, HALF>(w, h, x, vocab, hidden, k_tok, part, out, s); break;
        case 7: case 8: if constexpr (kLong) return launch_lm_t<8, MODE, false, 1, HALF>(w, h, x, vocab, hidden, k_tok, part, out, s); break;
        case 9: if constexpr (kLong) return launch_lm_t<9, MODE, false, 1, HALF>(w, h, x, vocab, hidden, k_tok, part, out, s); break;
        default: break;
    }
    return hipErrorInvalidValue;
}

// tokens [0, k_tok) with k_tok <= 16; `part` holds kLmMaxWorkgroups * 16 candidates
hipError_t launch_lm_head(const uint16_t* w, const float* h, int vocab, int hidden, int k_tok, void* part_ws,
                          int32_t* token_ids, float* max_logit, float* logits, hipStream_t s) {
    const int n_wg = lm_workgroups((vocab + 15) / 16, true);
    LmCand* part = static_cast<LmCand*>(part_ws);
    const hipError_t e = launch_lm_cpw<kLmHead, true>(w, h, nullptr, vocab, hidden, k_tok, part, logits, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(lm_head_pick_kernel, dim3(1), dim3(1024), 0, s, part, n_wg, k_tok, token_ids, max_logit);
    return hipGetLastError();
}

// Eight rows a strip where every one of them still has a compute unit: 1536 rows are 96 strips of sixteen.  28 dense layers, hidden 1536, 5
// tokens: 1055 -> 989 us (down 11.2 -> 8.8 in the trace), and with q|k|v 981.  A plain linear gains on more than 2048 columns: 2048 x 8192 on
// 16 tokens 13.9 -> 12.1, 1536 x 8960 on 5 8.6 -> 7.9; 2048 x 2048 and smaller take the launch either way, and keep sixteen.
static bool lm_half_strips(int n_out) { return (n_out + 7) / 8 <= device_cu_count(); }

// y[t][n] = sum_c W[n][c] x[t][c] for a dense row-major bf16 matrix and tokens [0, k_tok); every entry of y written
// (final values: the contraction is added up inside the workgroup).  k_in a multiple of 128, <= 9216.  A pass takes 16
// tg tokens: two groups where dense_stream_pair_ok(k_in), whose activations then fit the registers next to each other; more
// tokens are further passes of the same launch (the grid's second dimension).
hipError_t launch_dense_stream_linear(const uint16_t* w, const uint16_t* x, int n_out, int k_in, int k_tok, float* y, int tg,
                                      hipStream_t s) {
    if (k_tok < 1 || k_tok > 64) return hipErrorInvalidValue;
    if (tg == 2) {
        if (!dense_stream_pair_ok(k_in)) return hipErrorInvalidValue;
        switch ((k_in / kLmChunkCols + kLmWaves - 1) / kLmWaves) {
            case 1: return launch_lm_t<1, kLmPlain, false, 2>(w, nullptr, x, n_out, k_in, k_tok, nullptr, y, s);
            case 2: return launch_lm_t<2, kLmPlain, false, 2>(w, nullptr, x, n_out, k_in, k_tok, nullptr, y, s);
            case 3: return launch_lm_t<3, kLmPlain, false, 2>(w, nullptr, x, n_out, k_in, k_tok, nullptr, y, s);
            case 4: return launch_lm_t<4, kLmPlain, false, 2>(w, nullptr, x, n_out, k_in, k_tok, nullptr, y, s);
            default: return hipErrorInvalidValue;
        }
    }
    if (k_tok <= 16 && k_in > 2048 && lm_half_strips(n_out)) return launch_lm_cpw<kLmPlain, false, true>(w, nullptr, x, n_out, k_in, k_tok, nullptr, y, s);
    return launch_lm_cpw<kLmPlain, false>(w, nullptr, x, n_out, k_in, k_tok, nullptr, y, s);
}

hipError_t launch_dense_stream_norm(const uint16_t* w, const float* h, int n_out, int k_in, int k_tok, float* y, hipStream_t s) {
    if (k_tok < 1 || k_tok > 16 || !dense_stream_norm_ok(k_in, k_tok)) return hipErrorInvalidValue;
    if (lm_half_strips(n_out)) return launch_lm_cpw<kLmPlain, true, true>(w, h, nullptr, n_out, k_in, k_tok, nullptr, y, s);
    return launch_lm_cpw<kLmPlain, true>(w, h, nullptr, n_out, k_in, k_tok, nullptr, y, s);
}

hipError_t launch_dense_stream_gated(const uint16_t* w, const uint16_t* x, const float* h, int n_out, int k_in, int k_tok, uint16_t* m_out,
                                     hipStream_t s) {
    if (k_tok < 1 || k_tok > 64 || !dense_stream_gated_ok(n_out, k_in)) return hipErrorInvalidValue;
    float* out = reinterpret_cast<float*>(m_out);
    if (x) return launch_lm_cpw<kLmGated, false>(w, nullptr, x, n_out, k_in, k_tok, nullptr, out, s);
    if (!dense_stream_norm_ok(k_in, k_tok)) return hipErrorInvalidValue;
    return launch_lm_cpw<kLmGated, true>(w, h, nullptr, n_out, k_in, k_tok, nullptr, out, s);
}

hipError_t launch_dense_stream_add(const uint16_t* w, const uint16_t* x, int n_out, int k_in, int k_tok, float* h, hipStream_t s) {
    if (k_tok < 1 || !dense_stream_add_ok(n_out, k_in, k_tok)) return hipErrorInvalidValue;
    if (lm_half_strips(n_out)) return launch_lm_cpw<kLmAdd, false, true>(w, nullptr, x, n_out, k_in, k_tok, nullptr, h, s);
    return launch_lm_cpw<kLmAdd, false>(w, nullptr, x, n_out, k_in, k_tok, nullptr, h, s);
}

hipError_t launch_dense_stream_attend_add(const uint16_t* w, const float* qkv, int n_heads, int n_kv, int n_out, int k_tok, float* h,
                                          hipStream_t s) {
    const int k_in = n_heads * 128, rep = n_heads / n_kv;
    if (k_tok < 1 || !dense_stream_attend_ok(n_heads, n_out, k_tok)) return hipErrorInvalidValue;
    const bool half = lm_half_strips(n_out);
#define SD2_ATT_CASE(C, M) \
    if ((n_heads + kLmWaves - 1) / kLmWaves == C && lm_att_slots(M) == few_slots(k_tok)) \
        return half ? launch_lm_t<C, M, false, 1, true>(w, qkv, nullptr, n_out, k_in, k_tok, nullptr, h, s, rep) \
                    : launch_lm_t<C, M, false, 1, false>(w, qkv, nullptr, n_out, k_in, k_tok, nullptr, h, s, rep)
    SD2_ATT_CASE(1, kLmAtt2);
    SD2_ATT_CASE(2, kLmAtt2);
    SD2_ATT_CASE(3, kLmAtt2);
    SD2_ATT_CASE(4, kLmAtt2);
    SD2_ATT_CASE(1, kLmAtt5);
    SD2_ATT_CASE(2, kLmAtt5);
#undef SD2_ATT_CASE
    return hipErrorInvalidValue;
}

}  // namespace sd2
