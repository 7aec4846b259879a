// libsd2 -- attention of many query rows at once on the matrix cores (gfx950), head_dim 128.
//
// The precision is that of fp32 arithmetic, as in the kernels that take one query row at a time: where both operands are
// fp32 the products run on the fp32 matrix instruction; where one operand is bf16 (the cache) the other is split into
// three bf16 terms of eight bits each -- 24 bits, nothing is dropped -- and each term is multiplied on the bf16
// instruction, whose products are exact and whose sums are fp32: three instructions of 16 clocks take the place of eight
// of 32.  That holds while all is finite: an infinity times a term that is zero is NaN, where fp32 has an infinity.  A score
// that is not finite is computed again in fp32.
#include <atomic>

#include "sd2_device.h"
#include "sd2_internal.h"

namespace sd2 {

constexpr int kAttD = 128;

// A row's weight for a position that it does not attend to is zero, and the matrix instruction multiplies it all the same:
// an infinity or NaN in a value of a later token would reach the earlier ones.  So a wavefront whose sums are not all finite
// adds them again on the vector ALU, attended positions only (nothing is paid for that while all is finite).
constexpr float kFloatMax = 3.402823466e38f;
__device__ __forceinline__ bool finite4(const f32x4& v) {
    return fabsf(v[0]) <= kFloatMax && fabsf(v[1]) <= kFloatMax && fabsf(v[2]) <= kFloatMax && fabsf(v[3]) <= kFloatMax;
}

// ------------------------------------------------------------------ among the call's own tokens (up to 64)
//
// Workgroup (head, 16 queries): keys and values 0 .. last query as fp32 in LDS (summed from the split-K partials on the way),
// wavefront w takes keys 16 w .. 16 w + 15 for the scores, four rows of the softmax and 32 dimensions of the output.
// What bounds it is the chain load -> scores -> softmax -> output of one workgroup, not the arithmetic.
constexpr int kInRow = kAttD + 4;  // row pitch in LDS: sixteen rows fall into different banks
constexpr int kInThreads = 256;

__global__ __launch_bounds__(kInThreads) void inflight_attention_wide_kernel(const float* __restrict__ part, int n_splits, int k_tok, int q_out,
                                                                            int kv_out, int rep, uint16_t* __restrict__ ctx) {
    extern __shared__ __attribute__((aligned(16))) float in_smem[];
    float* ks = in_smem;                 // [64][kInRow]
    float* vs = ks + 64 * kInRow;        // [64][kInRow]
    float* qs = vs + 64 * kInRow;        // [16][kInRow]
    float* sc = qs + 16 * kInRow;        // [16][68]
    const int head = blockIdx.x, qt = blockIdx.y, grp = head / rep;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, g = lane >> 4;
    const int n_out = q_out + 2 * kv_out, n_keys = 16 * (qt + 1);
    const size_t stride = (size_t)k_tok * n_out;
    // a thread owns 16-byte pieces tid & 31 of rows tid / 32, tid / 32 + 8, ...: everything in flight at once
    const int piece = 4 * (tid & 31), row0 = tid >> 5;
    f32x4 kr[8], vr[8], qr[2];
#pragma unroll
    for (int j = 0; j < 8; ++j) kr[j] = vr[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    qr[0] = qr[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < n_splits; ++s) {
        const float* p = part + (size_t)s * stride;
        f32x4 ka[8], va[8], qa[2];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = row0 + 8 * j;
            ka[j] = va[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (row < n_keys && row < k_tok) {
                const float* src = p + (size_t)row * n_out + q_out + grp * kAttD + piece;
                ka[j] = *reinterpret_cast<const f32x4*>(src);
                va[j] = *reinterpret_cast<const f32x4*>(src + kv_out);
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = 16 * qt + row0 + 8 * j;
            qa[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (row < k_tok) qa[j] = *reinterpret_cast<const f32x4*>(p + (size_t)row * n_out + head * kAttD + piece);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            kr[j] += ka[j];
            vr[j] += va[j];
        }
        qr[0] += qa[0];
        qr[1] += qa[1];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (row0 + 8 * j < n_keys) {
            *reinterpret_cast<f32x4*>(ks + (row0 + 8 * j) * kInRow + piece) = kr[j];
            *reinterpret_cast<f32x4*>(vs + (row0 + 8 * j) * kInRow + piece) = vr[j];
        }
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<f32x4*>(qs + (row0 + 8 * j) * kInRow + piece) = qr[j];
    __syncthreads();
    if (wave <= qt) {
        // the four lane groups take 32 dimensions each: the order of the contraction is free as long as both operands agree
        f32x4 acc0 = f32x4{0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
        const float* qp = qs + n * kInRow + 32 * g;
        const float* kp = ks + (16 * wave + n) * kInRow + 32 * g;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const f32x4 a = *reinterpret_cast<const f32x4*>(qp + 4 * i), b = *reinterpret_cast<const f32x4*>(kp + 4 * i);
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], acc1, 0, 0, 0);
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], acc1, 0, 0, 0);
        }
        const f32x4 s = (acc0 + acc1) * 0.08838834764831845f;  // 1 / sqrt(128)
#pragma unroll
        for (int v = 0; v < 4; ++v) sc[(4 * g + v) * 68 + 16 * wave + n] = s[v];
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {  // wavefront w: rows 4 w + v, lane = key
        const int row = 4 * wave + v, query = 16 * qt + row;
        const bool on = lane <= query;
        const float s = on ? sc[row * 68 + lane] : -3.0e38f;
        float mx = s;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        const float e = on ? expf(s - mx) : 0.f;
        float sum = e;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        sc[row * 68 + lane] = e / sum;
    }
    __syncthreads();
    f32x4 o0 = f32x4{0.f, 0.f, 0.f, 0.f}, o1 = o0;
    const float* vp = vs + 32 * wave + n;
    for (int j = 0; j < n_keys; j += 4) {  // 16x16x4: lane (n, g) brings key j + g
        const float p = sc[n * 68 + j + g];
        o0 = __builtin_amdgcn_mfma_f32_16x16x4f32(p, vp[(j + g) * kInRow], o0, 0, 0, 0);
        o1 = __builtin_amdgcn_mfma_f32_16x16x4f32(p, vp[(j + g) * kInRow + 16], o1, 0, 0, 0);
    }
    if (__any(!finite4(o0) || !finite4(o1))) {
        o0 = o1 = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < n_keys; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (j <= 16 * qt + 4 * g + v) {
                    const float p = sc[(4 * g + v) * 68 + j];
                    o0[v] += p * vp[j * kInRow];
                    o1[v] += p * vp[j * kInRow + 16];
                }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int query = 16 * qt + 4 * g + v;
        if (query < k_tok) {
            uint16_t* dst = ctx + (size_t)query * q_out + head * kAttD + 32 * wave + n;
            dst[0] = f32_to_bf16(o0[v]);
            dst[16] = f32_to_bf16(o1[v]);
        }
    }
}

hipError_t launch_inflight_attention_wide(const float* part, int n_splits, int k_tok, int q_out, int kv_out, int n_heads, int n_kv,
                                          uint16_t* ctx, hipStream_t s) {
    if (k_tok < 1 || k_tok > 64 || n_heads % n_kv) return hipErrorInvalidValue;
    constexpr size_t lds = (size_t)((64 + 64 + 16) * kInRow + 16 * 68) * sizeof(float);
    static std::atomic<bool> raised{false};  // once, at the first call (a warm-up call precedes any graph capture)
    if (!raised.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&inflight_attention_wide_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        raised.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(inflight_attention_wide_kernel, dim3((unsigned)n_heads, (unsigned)((k_tok + 15) / 16)), dim3(kInThreads), lds, s, part,
                       n_splits, k_tok, q_out, kv_out, n_heads / n_kv, ctx);
    return hipGetLastError();
}

// ------------------------------------------------------------------ over the key/value cache
//
// Workgroup (key/value head, 16 query rows): the rows are (token, query head of the group) pairs in that order, so a cache
// row is read once per sixteen of them.  A wavefront takes tiles of 32 positions: scores of the sixteen rows (keys straight
// from the cache as matrix operands), running maximum and sum per row (online softmax), weighted values.  The values of a
// tile go through the wavefront's LDS, where an operand needs eight positions of one dimension: four-byte reads, lane = a pair
// of dimensions, whose even and odd ones become two operands; a row pitch of 320 bytes and the assignment position = 4 e + g of the
// eight entries to the four lane groups put the sixty-four reads of an instruction into as many banks.  The wavefronts' results meet
// in LDS at the end.
constexpr int kCaWaves = 8;
constexpr int kCaVRow = 320;                             // bytes: the four rows that lanes read side by side fall into different banks
constexpr int kCaPRow = 36;                              // floats
constexpr int kCaWaveBytes = 32 * kCaVRow + 16 * kCaPRow * 4;
constexpr int kCaORow = kAttD + 4;
constexpr int kCaMergeBytes = kCaWaves * (16 * kCaORow + 32) * 4;
constexpr size_t kCaLds = kCaWaves * kCaWaveBytes > kCaMergeBytes ? kCaWaves * kCaWaveBytes : kCaMergeBytes;

// eight fp32 values as three bf16 operands whose sum is the value
__device__ __forceinline__ void split_bf16x3(const float (&x)[8], Frag (&t)[3]) {
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = x[e];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t w = pack_bf16(r[2 * e], r[2 * e + 1]);
            t[k].u[e] = w;
            r[2 * e] -= __uint_as_float(w << 16);
            r[2 * e + 1] -= __uint_as_float(w & 0xffff0000u);
        }
}

// maximum over the sixteen lanes of a row, in every one of them
__device__ __forceinline__ float row_max(float v) {
#define SD2_ROW_MAX(ctrl) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true)))
    SD2_ROW_MAX(0x121);  // row_ror:1
    SD2_ROW_MAX(0x122);  // row_ror:2
    SD2_ROW_MAX(0x124);  // row_ror:4
    SD2_ROW_MAX(0x128);  // row_ror:8
#undef SD2_ROW_MAX
    return v;
}

__global__ __launch_bounds__(64 * kCaWaves) void cached_attention_wide_kernel(const float* __restrict__ q_rot, const uint16_t* __restrict__ k_cache,
                                                                             const uint16_t* __restrict__ v_cache, int max_pos, int pos0,
                                                                             int k_tok, int q_out, int rep, uint16_t* __restrict__ ctx) {
    extern __shared__ __attribute__((aligned(16))) uint8_t ca_smem[];
    const int grp = blockIdx.x, row_lo = 16 * blockIdx.y, n_rows = rep * k_tok;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n = lane & 15, g = lane >> 4;
    uint8_t* vbuf = ca_smem + wave * kCaWaveBytes;
    float* pbuf = reinterpret_cast<float*>(vbuf + 32 * kCaVRow);
    const uint16_t* kg = k_cache + (size_t)grp * max_pos * kAttD;
    const uint16_t* vg = v_cache + (size_t)grp * max_pos * kAttD;
    const int n_pos = pos0 + min(row_lo + 15, n_rows - 1) / rep + 1;  // positions any of the rows attends to

    // The first tile's keys and values are requested in front of the queries, every further tile's as soon as the tile before it has left
    // the registers (keys when its scores are there, values when they are in LDS): its trip to memory passes beside the softmax.
    Frag kf[2][4];
    u32x4 vr[8];
    auto request_tile = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const uint16_t* src = kg + (size_t)min(base + 16 * b + n, n_pos - 1) * kAttD + 8 * g;
#pragma unroll
            for (int i = 0; i < 4; ++i) kf[b][i].q = *reinterpret_cast<const u32x4*>(src + 32 * i);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) vr[i] = *reinterpret_cast<const u32x4*>(vg + (size_t)min(base + 4 * i + g, n_pos - 1) * kAttD + 8 * n);
    };
    request_tile(32 * wave);

    // operand A of the scores: row n, dimensions 32 i + 8 g + 0..7 (rows past the last repeat it; never written)
    Frag q[4][3];
    {
        const int row = min(row_lo + n, n_rows - 1), t = row / rep, r = row - t * rep;
        const float* src = q_rot + (size_t)t * q_out + ((size_t)grp * rep + r) * kAttD + 8 * g;
        f32x4 raw[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            raw[i][0] = *reinterpret_cast<const f32x4*>(src + 32 * i);
            raw[i][1] = *reinterpret_cast<const f32x4*>(src + 32 * i + 4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = raw[i][e >> 2][e & 3] * 0.08838834764831845f;  // 1 / sqrt(128)
            split_bf16x3(x, q[i]);
        }
    }
    int last[4];  // last position of the rows 4 g + v whose results this lane holds
#pragma unroll
    for (int v = 0; v < 4; ++v) last[v] = pos0 + min(row_lo + 4 * g + v, n_rows - 1) / rep;
    // scores of the rows 4 g + v at position pos; kf: the sixteen positions' keys as matrix operands
    auto scores = [&](const Frag (&kf)[4], int pos) __attribute__((always_inline)) {
        f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 2; k >= 0; --k)  // small terms first
#pragma unroll
            for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q[i][k].v, kf[i].v, s, 0, 0, 0);
        bool finite = true;
#pragma unroll
        for (int v = 0; v < 4; ++v) finite = finite && (pos > last[v] || fabsf(s[v]) <= kFloatMax);
        if (__any(!finite)) {
            const uint16_t* key = kg + (size_t)min(pos, n_pos - 1) * kAttD;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = min(row_lo + 4 * g + v, n_rows - 1), t = row / rep, r = row - t * rep;
                const float* src = q_rot + (size_t)t * q_out + ((size_t)grp * rep + r) * kAttD;
                float dot = 0.f;
#pragma unroll 1
                for (int d = 0; d < kAttD; ++d) dot += src[d] * 0.08838834764831845f * __uint_as_float((uint32_t)key[d] << 16);
                s[v] = dot;
            }
        }
        return s;
    };

    float m[4], l[4];
    f32x4 o[8];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        m[v] = -3.0e38f;
        l[v] = 0.f;
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int base = 32 * wave; base < n_pos; base += 32 * kCaWaves) {
        f32x4 s[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) s[b] = scores(kf[b], base + 16 * b + n);
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(vbuf + (4 * i + g) * kCaVRow + 16 * n) = vr[i];
        if (base + 32 * kCaWaves < n_pos) request_tile(base + 32 * kCaWaves);
        float p[2][4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool on0 = base + n <= last[v], on1 = base + 16 + n <= last[v];
            float mx = fmaxf(on0 ? s[0][v] : -3.0e38f, on1 ? s[1][v] : -3.0e38f);
            mx = fmaxf(row_max(mx), m[v]);
            const float f = expf(m[v] - mx);
            m[v] = mx;
            p[0][v] = on0 ? expf(s[0][v] - mx) : 0.f;
            p[1][v] = on1 ? expf(s[1][v] - mx) : 0.f;
            l[v] = l[v] * f + p[0][v] + p[1][v];
#pragma unroll
            for (int d = 0; d < 8; ++d) o[d][v] *= f;
        }
        // weights from result layout (lane = position) to operand layout (lane = row, entry e = position 4 e + g)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) pbuf[(4 * g + v) * kCaPRow + 8 * (n & 3) + 4 * b + (n >> 2)] = p[b][v];
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        float w[8];
        *reinterpret_cast<f32x4*>(&w[0]) = *reinterpret_cast<const f32x4*>(pbuf + n * kCaPRow + 8 * g);
        *reinterpret_cast<f32x4*>(&w[4]) = *reinterpret_cast<const f32x4*>(pbuf + n * kCaPRow + 8 * g + 4);
        Frag wt[3];
        split_bf16x3(w, wt);
        // Two dimensions of a position per read: o[2 j] takes the even ones of dimensions 32 j .. 32 j + 31, o[2 j + 1] the odd ones
        // (a 16-bit read per dimension and position is twice the reads, and LDS was what the tile waited for).
        const uint8_t* vp = vbuf + g * kCaVRow + 4 * n;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t pair[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) pair[e] = *reinterpret_cast<const uint32_t*>(vp + 4 * e * kCaVRow + 64 * j);
            Frag even, odd;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                even.u[e] = __builtin_amdgcn_perm(pair[2 * e + 1], pair[2 * e], 0x05040100u);
                odd.u[e] = __builtin_amdgcn_perm(pair[2 * e + 1], pair[2 * e], 0x07060302u);
            }
#pragma unroll
            for (int k = 2; k >= 0; --k) {
                o[2 * j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[k].v, even.v, o[2 * j], 0, 0, 0);
                o[2 * j + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[k].v, odd.v, o[2 * j + 1], 0, 0, 0);
            }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();  // the next tile overwrites both buffers
    }
    bool finite = true;
#pragma unroll
    for (int d = 0; d < 8; ++d) finite = finite && finite4(o[d]);
    if (__any(!finite)) {  // maxima and sums stand: they come from attended scores only
#pragma unroll
        for (int d = 0; d < 8; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int base = 32 * wave; base < n_pos; base += 32 * kCaWaves) {
            const int n_here = min(32, n_pos - base);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const uint16_t* src = kg + (size_t)min(base + 16 * b + n, n_pos - 1) * kAttD + 8 * g;
                Frag kf[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) kf[i].q = *reinterpret_cast<const u32x4*>(src + 32 * i);
                const f32x4 s = scores(kf, base + 16 * b + n);
#pragma unroll
                for (int v = 0; v < 4; ++v) pbuf[(4 * g + v) * kCaPRow + 16 * b + n] = expf(s[v] - m[v]);
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_wave_barrier();
            for (int j = 0; j < n_here; ++j) {
                const uint16_t* src = vg + (size_t)(base + j) * kAttD + 2 * n;
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const float x = __uint_as_float((uint32_t)src[32 * (d >> 1) + (d & 1)] << 16);
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (base + j <= last[v]) o[d][v] += pbuf[(4 * g + v) * kCaPRow + j] * x;
                }
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    float* om = reinterpret_cast<float*>(ca_smem);       // [waves][16][kCaORow]
    float* mm = om + kCaWaves * 16 * kCaORow;            // [waves][16] maxima, then [waves][16] sums
    float* ll = mm + kCaWaves * 16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float t = l[v];
        t += __shfl_xor(t, 1);
        t += __shfl_xor(t, 2);
        t += __shfl_xor(t, 4);
        t += __shfl_xor(t, 8);
        if (n == 0) {
            mm[wave * 16 + 4 * g + v] = m[v];
            ll[wave * 16 + 4 * g + v] = t;
        }
#pragma unroll
        for (int d = 0; d < 8; ++d) om[(wave * 16 + 4 * g + v) * kCaORow + 32 * (d >> 1) + 2 * n + (d & 1)] = o[d][v];
    }
    __syncthreads();
    const int mr = tid >> 5, d4 = 4 * (tid & 31), row = row_lo + mr;  // 512 threads: 16 rows of 32 pieces
    float gm = -3.0e38f, den = 0.f;
#pragma unroll
    for (int w = 0; w < kCaWaves; ++w) gm = fmaxf(gm, mm[w * 16 + mr]);
    f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kCaWaves; ++w) {
        const float f = expf(mm[w * 16 + mr] - gm);
        den += f * ll[w * 16 + mr];
        num += f * *reinterpret_cast<const f32x4*>(om + (w * 16 + mr) * kCaORow + d4);
    }
    if (row < n_rows) {
        const int t = row / rep, r = row - t * rep;
        const float inv = 1.0f / den;
        *reinterpret_cast<uint2*>(ctx + (size_t)t * q_out + ((size_t)grp * rep + r) * kAttD + d4) =
            make_uint2(pack_bf16(num[0] * inv, num[1] * inv), pack_bf16(num[2] * inv, num[3] * inv));
    }
}

hipError_t launch_cached_attention_wide(const float* q_rot, const uint16_t* k_cache, const uint16_t* v_cache, int max_pos, int pos0, int k_tok,
                                        int q_out, int n_heads, int n_kv, uint16_t* ctx, hipStream_t s) {
    static std::atomic<bool> raised{false};
    if (!raised.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&cached_attention_wide_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCaLds);
        if (e != hipSuccess) return e;
        raised.store(true, std::memory_order_release);
    }
    const int rep = n_heads / n_kv;
    hipLaunchKernelGGL(cached_attention_wide_kernel, dim3((unsigned)n_kv, (unsigned)((rep * k_tok + 15) / 16)), dim3(64 * kCaWaves), kCaLds, s,
                       q_rot, k_cache, v_cache, max_pos, pos0, k_tok, q_out, rep, ctx);
    return hipGetLastError();
}

}  // namespace sd2
