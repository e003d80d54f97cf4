// linattn_common.hpp -- shared pieces of the linear-attention kernels: the
// register layouts of 16-row blocks, LDS staging of 64-row chunks, the
// contractions on v_mfma_f32_16x16x4_f32, phi.
//
// A workgroup of four wavefronts owns a segment of consecutive 64-row chunks
// of one head and walks it with the 64x64 state in registers, a quarter of its
// columns per wavefront.  A chunk is four 16-row blocks: wavefront w forms
// the causal products of block w alone, and all four then take the blocks in
// order against their quarter of the state.
//
// With lane = 16 g + c (g = 0..3, c = 0..15), v_mfma_f32_16x16x4_f32 takes
// A[i = c][k = g], B[k = g][j = c] and returns D[i = 4 g + r][j = c] in
// register r.  A block M[t][col] is read from LDS in three layouts:
//   row fragment  RF[r].s = M[t = c][col = 16 r + 4 g + s]
//   col fragment  CF[q].s = M[t = 4 g + q][col = cm(c) + s],
//                 cm(c) = 16 (c & 3) + 4 (c >> 2)
//   slice         SL.q    = M[t = 4 g + q][col = 16 w + c]   (wavefront w)
// (RF and CF are 16-byte reads, SL 4-byte; none meets a bank conflict at a row
// stride of 68 floats.)  A contraction over columns takes row fragments on
// both sides (k-slot g of MFMA (r, s) is column 16 r + 4 g + s), a contraction
// over rows column fragments and slices (k-slot g of MFMA q is row 4 g + q).
// Results arrive where the next product wants them:
//   * X Y^T of row fragments is returned as [row 4 g + r of X][row c of Y],
//     the B operand of MFMA q = r of a contraction over X's rows;
//   * the state quarter X^T Y (A = X CF.s, B = Y SL) is returned as
//     st[s][r] = [X column 16 r + 4 g + s][Y column 16 w + c], since
//     cm(4 g + r) = 16 r + 4 g: the A operand of MFMA (r, s) of a contraction
//     over X's columns against a row fragment;
//   * both contractions against a state or a slice return output column
//     16 w + 4 g + r of row c in register r: one 16-byte store per lane.
#pragma once

#include "scan_common.hpp"
#include "kernels.hpp"

namespace memoroid {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDim = 64;                          // head width
constexpr int kChunk = kLinChunkRows;             // rows per chunk
constexpr int kBlk = 16;                          // rows per block
constexpr int kLD = 68;                           // LDS row stride in floats (16-byte aligned rows)
constexpr int kTileF = kChunk * kLD;              // floats of a staged chunk
constexpr int kStateWords = kLinStateWords;       // S (64x64, row kd) followed by z (64)

// phi(u) = 1 + ELU(u): u + 1 for u > 0, exp(u) otherwise.  exp uses the
// hardware base-2 exponential (relative error a few ulp, far inside the fp32
// tolerance of the readout).
__device__ __forceinline__ float phi(float u) { return u > 0.0f ? u + 1.0f : __expf(u); }
// phi'(u) from phi(u): 1 for u > 0 (phi = u + 1 >= 1), exp(u) = phi(u) <= 1
// otherwise, i.e. min(phi(u), 1), bit for bit; a NaN stays NaN
__device__ __forceinline__ float phi_prime_of_phi(float ph) { return ph > 1.0f ? 1.0f : ph; }
__device__ __forceinline__ f32x4 phi4(f32x4 v) { return f32x4{phi(v.x), phi(v.y), phi(v.z), phi(v.w)}; }
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }

typedef f32x4 Frag[4];

struct LinLane {
    int tid, lane, w, g, c, cm;
    __device__ LinLane() {
        tid = threadIdx.x;
        lane = tid & 63;
        w = __builtin_amdgcn_readfirstlane(tid >> 6);
        g = lane >> 4;
        c = lane & 15;
        cm = 16 * (c & 3) + 4 * (c >> 2);
    }
};

// ------------------------------------------------------------ global memory
// Rows t0 .. t0 + 63 of one head of a [T][H][64] tensor as a buffer resource;
// rows at or past T (and every row when `have` is false) read as zeros and
// drop their stores.
struct ChunkRows {
    Rsrc r;
    uint32_t row_bytes;
    __device__ __forceinline__ f32x4 load(int row, int col) const {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)((uint32_t)row * row_bytes + 4u * col), 0, 0);
        return f32x4{__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
    }
    __device__ __forceinline__ float load1(int row, int col) const {
        return __uint_as_float(
            __builtin_amdgcn_raw_buffer_load_b32(r, (int)((uint32_t)row * row_bytes + 4u * col), 0, 0));
    }
    // outputs are written once and read by no later kernel: non-temporal
    __device__ __forceinline__ void store_nt(int row, int col, f32x4 v) const {
        const u32x4 w = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
        __builtin_amdgcn_raw_buffer_store_b128(w, r, (int)((uint32_t)row * row_bytes + 4u * col), 0, kNt);
    }
};
__device__ __forceinline__ ChunkRows chunk_rows(const float* p, int64_t t0, int64_t T, int64_t H, int64_t h,
                                                bool have = true) {
    const int64_t left = T - t0;
    const int64_t n = !have || left <= 0 ? 0 : (left < kChunk ? left : kChunk);
    return ChunkRows{make_rsrc(p + (t0 * H + h) * kDim, n > 0 ? ((n - 1) * H + 1) * kDim * 4 : 0),
                     (uint32_t)(H * kDim * 4)};
}
// one float per row from a [T][H] array, the same way
__device__ __forceinline__ ChunkRows row_scalars(const float* p, int64_t t0, int64_t T, int64_t H, int64_t h,
                                                 bool have = true) {
    const int64_t left = T - t0;
    const int64_t n = !have || left <= 0 ? 0 : (left < kChunk ? left : kChunk);
    return ChunkRows{make_rsrc(p + t0 * H + h, n > 0 ? ((n - 1) * H + 1) * 4 : 0), (uint32_t)(H * 4)};
}

// A chunk staged by the workgroup: thread `tid` holds row 16 u + tid / 16,
// columns 4 (tid % 16) .. + 3 for u = 0..3.
__device__ __forceinline__ void fetch_chunk(Frag& v, const ChunkRows& cr, const LinLane& L) {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = cr.load(16 * u + (L.tid >> 4), (L.tid & 15) * 4);
}
template <bool PHI>
__device__ __forceinline__ void stage_chunk(float* s, const Frag& v, const LinLane& L) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
        *(f32x4*)(s + (16 * u + (L.tid >> 4)) * kLD + (L.tid & 15) * 4) = PHI ? phi4(v[u]) : v[u];
}

// -------------------------------------------------------------- LDS layouts
__device__ __forceinline__ void lds_rf(Frag& v, const float* s, int row0, const LinLane& L) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = *(const f32x4*)(s + (row0 + L.c) * kLD + 16 * r + 4 * L.g);
}
__device__ __forceinline__ void lds_cf(Frag& v, const float* s, int row0, const LinLane& L) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = *(const f32x4*)(s + (row0 + 4 * L.g + q) * kLD + L.cm);
}
__device__ __forceinline__ f32x4 lds_slice(const float* s, int row0, const LinLane& L) {
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = s[(row0 + 4 * L.g + q) * kLD + 16 * L.w + L.c];
    return v;
}

// rows (4 g + q) for which bit t of `rows` is clear become zeros (a select, so
// non-finite values there never enter)
__device__ __forceinline__ void select_rows(Frag& v, uint32_t rows, const LinLane& L) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool in = (rows >> (4 * L.g + q)) & 1u;
#pragma unroll
        for (int s = 0; s < 4; ++s) v[q][s] = in ? v[q][s] : 0.0f;
    }
}
__device__ __forceinline__ void select_rows(f32x4& v, uint32_t rows, const LinLane& L) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = (rows >> (4 * L.g + q)) & 1u ? v[q] : 0.0f;
}

// ------------------------------------------------------------- contractions
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// sum over the 64 columns of x and y (row fragments): register r holds
// [row 4 g + r of x][row c of y].  Two chains, added at the end.
__device__ __forceinline__ f32x4 mul_rows(const Frag& x, const Frag& y) {
    f32x4 d0 = zero4(), d1 = zero4();
#pragma unroll
    for (int r = 0; r < 4; r += 2)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            d0 = mfma4(x[r][s], y[r][s], d0);
            d1 = mfma4(x[r + 1][s], y[r + 1][s], d1);
        }
    return d0 + d1;
}
// the state quarter times a row fragment; st[s][r] is an A operand like
// y[r][s] a B operand.  Register r: column 16 w + 4 g + r of row c.
__device__ __forceinline__ f32x4 mul_state(const Frag& st, const Frag& y) {
    f32x4 d0 = zero4(), d1 = zero4();
#pragma unroll
    for (int r = 0; r < 4; r += 2)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            d0 = mfma4(st[s][r], y[r][s], d0);
            d1 = mfma4(st[s][r + 1], y[r + 1][s], d1);
        }
    return d0 + d1;
}
// st += x^T y over a block's rows (x a column fragment, y a slice)
__device__ __forceinline__ void state_add(Frag& st, const Frag& x, const f32x4& y) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int s = 0; s < 4; ++s) st[s] = mfma4(x[q][s], y[q], st[s]);
}
// The same, with the block's sum formed on its own and added once: a state that
// a long episode has made large then takes one rounding per block instead of
// one per row.  The gradient needs that (dq and dk subtract two nearly equal
// products of such states): without it their errors against 64 bits grew with
// the episode, 3.8e-7 and 2.1e-7 at 1000 steps, 8.3e-7 and 4.6e-7 at 262144;
// with it 4.3e-7 and 2.2e-7 there.  Two of the four sums at a time, for the
// registers.  T = 32768, 4 heads: gradient 152.4 -> 154.2 us.
__device__ __forceinline__ void state_add_once(Frag& st, const Frag& x, const f32x4& y) {
#pragma unroll
    for (int s = 0; s < 4; s += 2) {
        f32x4 d0 = zero4(), d1 = zero4();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            d0 = mfma4(x[q][s], y[q], d0);
            d1 = mfma4(x[q][s + 1], y[q], d1);
        }
        st[s] += d0;
        st[s + 1] += d1;
    }
}
// acc += sum over t of p[t][c] x[t][16 w + .], p[q] the weight of row 4 g + q
__device__ __forceinline__ f32x4 mul_slice(const f32x4& x, const f32x4& p, f32x4 acc) {
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = mfma4(x[q], p[q], acc);
    return acc;
}
// The same, with row t taken only where bit t of the lane's `keep` is set.
// A slice holding a value that is not finite would carry it through the zeros
// of p (0 * NaN), so each of the 16 targets then takes its own copy of x with
// the other rows selected to zeros.
__device__ __forceinline__ f32x4 mul_slice_kept(const f32x4& x, const f32x4& p, uint32_t keep, f32x4 acc,
                                                const LinLane& L) {
    float z = 0.0f;                        // stays zero while every value is finite
#pragma unroll
    for (int q = 0; q < 4; ++q) z = __builtin_fmaf(x[q], 0.0f, z);
    if (__ballot(z != 0.0f) == 0) return mul_slice(x, p, acc);
#pragma unroll 1
    for (int c0 = 0; c0 < kBlk; ++c0) {
        const uint32_t rows = (uint32_t)__builtin_amdgcn_readlane((int)keep, c0);
        f32x4 xs = x;
        select_rows(xs, rows, L);
        const f32x4 part = mul_slice(xs, p, zero4());
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] += L.c == c0 ? part[r] : 0.0f;
    }
    return acc;
}

// sum over the four lanes that share c
__device__ __forceinline__ float sum_g(float v) {
    v += lanes_xor(v, 16);
    v += lanes_xor(v, 32);
    return v;
}
// column sums of a column fragment, row 4 g + q weighted by w[q]: columns
// cm(c) .. + 3, the same in every g
__device__ __forceinline__ f32x4 col_sums(const Frag& x, const f32x4& w) {
    f32x4 s = zero4();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = __builtin_fmaf(w[q], x[q][e], s[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = sum_g(s[e]);
    return s;
}
__device__ __forceinline__ float dot_frag(const Frag& a, const Frag& b) {
    f32x4 s = zero4();
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = __builtin_fmaf(a[r][e], b[r][e], s[e]);
    return (s.x + s.y) + (s.z + s.w);
}
__device__ __forceinline__ f32x4 select4(bool c, f32x4 v) {
    return f32x4{c ? v.x : 0.0f, c ? v.y : 0.0f, c ? v.z : 0.0f, c ? v.w : 0.0f};
}
// the state z of the next block: z restarts from the block's own sums when the
// block holds a begin step
__device__ __forceinline__ f32x4 z_then(f32x4 z, uint32_t begins, f32x4 own) {
    return begins ? own : z + own;
}

// -------------------------------------------------------------- begin flags
// Begin bits of a chunk's 64 rows.  Rows at or past T count as begins: each is
// an episode of its own, so nothing of them reaches a real row and no other
// bound check is needed.
__device__ __forceinline__ uint32_t fetch_flag(const uint8_t* start, int64_t t0, int64_t T) {
    return bload_u8(make_rsrc(start + t0, T - t0), threadIdx.x & 63);
}
__device__ __forceinline__ uint64_t begin_bits(uint32_t flag, int64_t t0, int64_t T) {
    const int64_t t = t0 + (threadIdx.x & 63);
    return __ballot(t >= T || t == 0 || flag != 0u);
}
__device__ __forceinline__ uint32_t block_bits(uint64_t m, int b) { return (uint32_t)(m >> (16 * b)) & 0xFFFFu; }
// first row of row t's episode inside the block (0 when it began earlier), and
// one past its last row inside the block
__device__ __forceinline__ int first_of(uint32_t begins, int t) {
    const uint32_t m = begins & ((2u << t) - 1u);
    return m ? 31 - __builtin_clz(m) : 0;
}
__device__ __forceinline__ int end_of(uint32_t begins, int t) {
    const uint32_t m = begins & ~((2u << t) - 1u);
    return m ? __builtin_ctz(m) : kBlk;
}
__device__ __forceinline__ uint32_t bit_range(int lo, int hi) {      // bits lo .. hi - 1, 0 <= lo <= hi <= 16
    return ((1u << hi) - 1u) & ~((1u << lo) - 1u);
}

// ------------------------------------------------------------ segment states
// A segment's state words in memory (S[kd][n] row-major, then z) as a buffer;
// an absent one reads as zeros.
__device__ __forceinline__ Rsrc state_rows(const float* states, int64_t seg, int64_t H, int64_t h, bool have) {
    return make_rsrc(states + (have ? (seg * H + h) * kStateWords : 0), have ? kStateWords * 4 : 0);
}
__device__ __forceinline__ f32x4 bload4(Rsrc r, uint32_t off) {
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    return f32x4{__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w)};
}
// st[s][r] = S[16 r + 4 g + s][16 w + c]: the state against phi row fragments
__device__ __forceinline__ void load_state_kd(Frag& st, Rsrc rs, const LinLane& L) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int s = 0; s < 4; ++s)
            st[s][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rs, ((16 * r + 4 * L.g + s) * kDim + 16 * L.w + L.c) * 4, 0, 0));
}
// st[s][r] = S[16 w + c][16 r + 4 g + s]: the state against value row fragments
__device__ __forceinline__ void load_state_n(Frag& st, Rsrc rs, const LinLane& L) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const f32x4 v = bload4(rs, (uint32_t)((16 * L.w + L.c) * kDim + 16 * r + 4 * L.g) * 4u);
#pragma unroll
        for (int s = 0; s < 4; ++s) st[s][r] = v[s];
    }
}
// The state before segment `seg` (REV: after it): load(rs) reads the
// neighbour's scanned state or, DIRECT (at most kLinDirectSegs segments), its
// summary, to which add(rs) adds the others back to the nearest segment that
// holds a begin step, found with one ballot over the flags.
template <bool DIRECT, bool REV, class Load, class Add>
__device__ __forceinline__ void state_before(const float* states, const uint8_t* R, int64_t seg, int64_t nseg, int64_t H,
                                             int64_t h, Load&& load, Add&& add) {
    const bool any = REV ? seg + 1 < nseg : seg > 0;
    const int64_t near = REV ? seg + 1 : seg - 1;
    load(state_rows(states, near, H, h, any));
    if (!DIRECT || !any) return;
    const uint32_t fl = bload_u8(make_rsrc(R, nseg), threadIdx.x & 63);
    const uint64_t holds = __ballot(fl != 0u);          // segments with a begin step
    const uint64_t m = REV ? holds & ~((1ull << near) - 1ull) : holds & ((2ull << near) - 1ull);
    const int far = m ? (REV ? __builtin_ctzll(m) : 63 - __builtin_clzll(m)) : (REV ? (int)nseg - 1 : 0);
    const int more = REV ? far - (int)near : (int)near - far;
#pragma unroll 2
    for (int i = 1; i <= more; ++i) add(state_rows(states, REV ? near + i : near - i, H, h, true));
}
__device__ __forceinline__ void add_frag(Frag& a, const Frag& b) {
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] += b[s];
}
__device__ __forceinline__ float state_z1(Rsrc rs, int i) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (kDim * kDim + i) * 4, 0, 0));
}
__device__ __forceinline__ f32x4 state_z4(Rsrc rs, int i) { return bload4(rs, (uint32_t)(kDim * kDim + i) * 4u); }
__device__ __forceinline__ void store_state_n(float* p, const Frag& st, const LinLane& L) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
        *(f32x4*)(p + (16 * L.w + L.c) * kDim + 16 * r + 4 * L.g) = f32x4{st[0][r], st[1][r], st[2][r], st[3][r]};
}

}  // namespace memoroid
