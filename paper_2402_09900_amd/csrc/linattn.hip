// linattn.hip -- kernels of the linear-transformer memoroid (App. G.1) over a
// tape with resets, for gfx950.
//
// The memoroid's monoid is a plain sum, (S, z) . (S', z') = (S + S', z + z'),
// of outer products phi(k) v^T and of phi(k); under the reset transform the
// state of step t sums only the steps of t's episode up to t.  The tape is cut
// into segments of a few 64-row chunks (lin_chunks in abi.hip), and a workgroup
// takes one segment of one head:
//
//   summary kernel: dS = sum of phi(k) v^T and dz = sum of phi(k) over the
//     rows from the segment's last begin step on; R = "segment holds a begin";
//   state scan: the segment states are scanned with resets, in place, giving
//     the state after every segment;
//   output kernel: walks the segment's chunks with the state in registers.
//     Per 16-row block, with first(i) the first row of row i's episode in the
//     block and the state taking part only in rows before the block's first
//     begin:
//       A   = phi(Q) phi(K)^T,  masked to first(i) <= j <= i
//       out = (A V + phi(Q) S) / (rowsum(A) + phi(Q) z)
//     and S += phi(K)^T V, z += sum phi(K) over the rows from the last begin;
//     the head-0 workgroups also produce the episode index of their steps.
//
// Blocks of 16 rows do fewer flops than whole 64-row chunks would (the causal
// product costs 16 columns a row instead of 40), and a segment of several
// chunks writes and reads fewer states (16.6 KB each).  See linattn_common.hpp
// for the layouts that let a block's products and the state meet in registers.
//
// Measured against one workgroup per 64-row chunk with every chunk's state
// through memory and a look-back scan over them (T = 32768, 4 heads, calls one
// after another): forward 72 -> 66 us, gradient 196 -> 154 us; T = 1000: 21 -> 18
// and 45 -> 37 us.  Kernels in a trace over several sets of buffers (T = 32768):
// summary 23 -> 21, scan 15 -> 6.6, output 49 -> 46 us.
#include "linattn_common.hpp"

namespace memoroid {

// ---------------------------------------------------------------- summaries
// Bound by instruction issue and its fixed start and end (19 us at T = 32768,
// 4 heads, no fewer with every load served by the L2; its reads take 11 us at
// copy speed and its MFMAs 7).
__global__ __launch_bounds__(256, 4) void linattn_summary_kernel(LinSummaryArgs p) {
    __shared__ __attribute__((aligned(16))) float sV[2][kTileF];
    const int64_t seg = blockIdx.x, h = blockIdx.y;
    const LinLane L;
    // header and episode-index count words, prepared (all-ones bytes, and the
    // call's signature in the header) for the later kernels (stream order)
    {
        const int64_t nblk = (int64_t)gridDim.x * gridDim.y;
        const int64_t gid = (int64_t)(blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
        const u32x4 ones = {kEmpty32, kEmpty32, kEmpty32, kEmpty32};
        static_assert(offsetof(WsHeader, sig) == 8, "the signature is the second half of the first unit");
        const u32x4 head = {kEmpty32, kEmpty32, (uint32_t)p.sig, (uint32_t)(p.sig >> 32)};
        for (int64_t i = gid; i < p.fill16; i += nblk * 256) p.fill[i] = i == 0 ? head : ones;
    }
    const int64_t seg0 = seg * p.chunks * kChunk;
    // V goes through LDS (every wavefront takes all of its columns), the
    // wavefront's 16 columns of K straight to registers; a chunk ahead, K block
    // by block as the registers become free
    Frag vreg, kreg;
    uint32_t flag;
    auto fetch_v = [&](int ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const bool have = ch < p.chunks;
        flag = fetch_flag(p.start, have ? t0 : 0, have ? p.T : 0);
        fetch_chunk(vreg, chunk_rows(p.v, t0, p.T, p.H, h, have), L);
    };
    auto fetch_k = [&](int ch, int b) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk + 16 * b;
        const ChunkRows ck = chunk_rows(p.k, t0, p.T, p.H, h, ch < p.chunks);
#pragma unroll
        for (int q = 0; q < 4; ++q) kreg[b][q] = ck.load1(4 * L.g + q, 16 * L.w + L.c);
    };
    fetch_v(0);
#pragma unroll
    for (int b = 0; b < 4; ++b) fetch_k(0, b);
    Frag st;                                   // st[s][r] = dS[16 w + c][16 r + 4 g + s]
#pragma unroll
    for (int s = 0; s < 4; ++s) st[s] = zero4();
    float z = 0.0f;                            // dz[16 w + c], this lane's rows
    bool any = false;
#pragma unroll 1
    for (int ch = 0; ch < p.chunks; ++ch) {
        float* const sv = sV[ch & 1];
        stage_chunk<false>(sv, vreg, L);
        const uint64_t m = begin_bits(flag, seg0 + (int64_t)ch * kChunk, p.T);
        any = any || m != 0;
        barrier_lds();
        fetch_v(ch + 1);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t mb = block_bits(m, b);
            Frag vc;
            lds_cf(vc, sv, 16 * b, L);
            f32x4 kc = phi4(kreg[b]);
            fetch_k(ch + 1, b);
            if (mb) {
                const uint32_t keep = bit_range(31 - __builtin_clz(mb), kBlk);
                select_rows(vc, keep, L);
                select_rows(kc, keep, L);
#pragma unroll
                for (int s = 0; s < 4; ++s) st[s] = zero4();
                z = 0.0f;
            }
            z += (kc.x + kc.y) + (kc.z + kc.w);
            state_add_once(st, vc, kc);
        }
    }
    float* const out = p.states + (seg * p.H + h) * kStateWords;
    store_state_n(out, st, L);
    z = sum_g(z);
    if (L.g == 0) out[kDim * kDim + 16 * L.w + L.c] = z;
    if (h == 0 && L.tid == 0) p.R[seg] = any ? 1 : 0;
}

// ---------------------------------------------------------------- state scan
// Segmented prefix sum of the segment states, in place, from the first
// segment on (REV: from the last back): y_s = x_s when segment s holds a begin
// step, else x_s + y_{s-1} (REV: y_{s+1}).  A workgroup takes one 128-byte line
// of the states (8 16-byte columns) and all segments, 32 RPT of them at a
// time: thread (grp, col) holds RPT consecutive segments of a column in
// registers, the 32 groups combine through LDS.  Loads go through a buffer
// resource, so the edges need no branches and all of them are in flight at
// once: the scan is one read and one write of the states (128 segments of 4
// heads 6.3 us, 512 segments 12.8 us = 5.3 TB/s; predicated pointer loads took
// 12 us on 256 segments against 8.6).
constexpr int kScanCols = 8, kScanGroups = kLinScanGroups;
template <int RPT, bool REV>
__global__ __launch_bounds__(256) void state_scan_kernel(LinScanArgs p) {
    __shared__ f32x4 s_tot[kScanGroups][kScanCols];
    __shared__ uint32_t s_flag[kScanGroups];
    static_assert(RPT <= kLinScanMaxRows, "kLinMaxHeads follows from the largest tile");
    constexpr int kTile = kScanGroups * RPT;
    const int col = threadIdx.x % kScanCols, grp = threadIdx.x / kScanCols;
    const uint32_t row_bytes = (uint32_t)(p.width * 4);
    const uint32_t c0 = (uint32_t)(blockIdx.x * kScanCols + col) * 16u;   // width is a multiple of 32 floats
    f32x4 carry = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int64_t base = 0; base < p.n; base += kTile) {
        // the tile's segments in memory order: s0 .. s0 + rows - 1; place l of
        // the scan order is segment l (REV: rows - 1 - l) among them
        const int rows = (int)(p.n - base < kTile ? p.n - base : kTile);
        const int64_t s0 = REV ? p.n - base - rows : base;
        const Rsrc rs = make_rsrc(p.states + s0 * p.width, (int64_t)rows * row_bytes);
        const Rsrc rr = make_rsrc(p.R + s0, rows);
        f32x4 x[RPT];
        uint32_t fl[RPT], off[RPT];
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int l = grp * RPT + i;
            const int s = REV ? rows - 1 - l : l;
            off[i] = l < rows ? (uint32_t)s * row_bytes + c0 : kOob;
            fl[i] = bload_u8(rr, l < rows ? (uint32_t)s : kOob);
            x[i] = bload4(rs, off[i]);
        }
        uint32_t flag = 0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) flag |= (fl[i] != 0u ? 1u : 0u) << i;
        f32x4 tot = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < RPT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[e] = (flag >> i) & 1u ? x[i][e] : tot[e] + x[i][e];
        __syncthreads();                               // the last round's totals have been read
        s_tot[grp][col] = tot;
        if (col == 0) s_flag[grp] = flag != 0u;
        __syncthreads();
        f32x4 y = carry;
#pragma unroll 8
        for (int k = 0; k < kScanGroups; ++k) {
            const f32x4 t = s_tot[k][col];
            const bool f = s_flag[k] != 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                carry[e] = f ? t[e] : carry[e] + t[e];
                y[e] = k + 1 == grp ? carry[e] : y[e];    // the state before this thread's run
            }
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (flag >> i) & 1u ? x[i][e] : y[e] + x[i][e];
            const u32x4 w = {__float_as_uint(y.x), __float_as_uint(y.y), __float_as_uint(y.z), __float_as_uint(y.w)};
            __builtin_amdgcn_raw_buffer_store_b128(w, rs, (int)off[i], 0, 0);
        }
    }
}

// ------------------------------------------------------------------- output

// Three workgroups' registers per CU; at T = 32768 and 4 heads the grid has two
// per CU, MFMAs keep the matrix cores 43 % busy, counted (43 us in a trace, 17 us
// of MFMA and 25 us of traffic), the rest being the phases of a chunk (staging,
// A of the own block, z and den) that two wavefronts per SIMD only partly
// overlap.  Loading V a phase earlier (2 us slower) or a branch-free path for
// chunks without begin steps (the same time) gained nothing.
template <bool DIRECT>
__global__ __launch_bounds__(256, 3) void linattn_output_kernel(LinOutputArgs p) {
    __shared__ __attribute__((aligned(16))) float sQ[kTileF];     // phi(Q)
    __shared__ __attribute__((aligned(16))) float sK[kTileF];     // phi(K)
    __shared__ f32x4 sA[4][64];                                   // each block's masked A, as mul_rows returns it
    __shared__ __attribute__((aligned(16))) float sZ[5][kDim];    // column sums of each block; [4]: z before the chunk
    __shared__ float sDen[kChunk];                                // 1 / den of the chunk's rows
    const int64_t seg = blockIdx.x, h = blockIdx.y;
    const LinLane L;
    const int64_t seg0 = seg * p.chunks * kChunk;
    const int64_t left = (p.T - seg0 + kChunk - 1) / kChunk;
    const int nch = (int)(left < p.chunks ? left : p.chunks);

    Frag qreg, kreg, vreg;                     // next chunk; vreg[b]: slices of V
    uint32_t flag;
    auto fetch_qk = [&](int ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const bool have = ch < nch;
        flag = fetch_flag(p.start, have ? t0 : 0, have ? p.T : 0);
        fetch_chunk(kreg, chunk_rows(p.k, t0, p.T, p.H, h, have), L);
        fetch_chunk(qreg, chunk_rows(p.q, t0, p.T, p.H, h, have), L);
    };
    auto fetch_v = [&](int ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const ChunkRows cv = chunk_rows(p.v, t0, p.T, p.H, h, ch < nch);
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) vreg[b][q] = cv.load1(16 * b + 4 * L.g + q, 16 * L.w + L.c);
    };
    fetch_qk(0);
    Frag st;                                   // st[s][r] = S[16 r + 4 g + s][16 w + c]
    float z_in = 0.0f;
    state_before<DIRECT, false>(
        p.states, p.R, seg, p.nseg, p.H, h,
        [&](Rsrc rs) {
            load_state_kd(st, rs, L);
            z_in = state_z1(rs, L.lane);
        },
        [&](Rsrc rs) {
            Frag s;
            load_state_kd(s, rs, L);
            z_in += state_z1(rs, L.lane);
            add_frag(st, s);
        });
    fetch_v(0);
    if (L.w == 0) sZ[4][L.lane] = z_in;

    // episode index (head-0 workgroups): wavefront 2 publishes the segment's
    // own begin count at once; wavefront 1 looks up the count before it when
    // the outputs are done
    const bool want_idx = p.idx != nullptr && h == 0;
    if (want_idx && L.w == 2) {
        uint32_t own = 0;
        for (int ch = 0; ch < nch; ++ch) {
            const int64_t t0 = seg0 + (int64_t)ch * kChunk;
            const int64_t t = t0 + L.lane;
            own += (uint32_t)__builtin_popcountll(
                __ballot(t < p.T && (t == 0 || fetch_flag(p.start, t0, p.T) != 0u)));
        }
        if (L.lane == 0) publish64(p.cnt + seg, (seg == 0 ? kCountIncl : kCountOwn) | own);
    }

#pragma unroll 1
    for (int ch = 0; ch < nch; ++ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const uint64_t m = begin_bits(flag, t0, p.T);
        stage_chunk<true>(sK, kreg, L);
        stage_chunk<true>(sQ, qreg, L);
        Frag vs;
#pragma unroll
        for (int b = 0; b < 4; ++b) vs[b] = vreg[b];
        barrier_lds();
        fetch_qk(ch + 1);

        // ---- block w alone: A and its row sums, the block's column sums of
        // phi(K) from its last begin on
        const uint32_t mw = block_bits(m, L.w);
        const int first = first_of(mw, L.c);
        const bool cont = (mw & ((2u << L.c) - 1u)) == 0u;       // row c's episode began before the block
        Frag qr;
        float den = 0.0f;
        {
            Frag kr;
            lds_rf(kr, sK, 16 * L.w, L);
            lds_rf(qr, sQ, 16 * L.w, L);
            f32x4 at = mul_rows(kr, qr);                          // phi(k_j) . phi(q_c), j = 4 g + r
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = 4 * L.g + r;
                at[r] = j <= L.c && j >= first ? at[r] : 0.0f;
                den += at[r];
            }
            sA[L.w][L.lane] = at;
            Frag kc;
            lds_cf(kc, sK, 16 * L.w, L);
            if (mw) select_rows(kc, bit_range(31 - __builtin_clz(mw), kBlk), L);
            const f32x4 zs = col_sums(kc, f32x4{1.0f, 1.0f, 1.0f, 1.0f});
            if (L.g == 0) *(f32x4*)(&sZ[L.w][L.cm]) = zs;
        }
        barrier_lds();
        float qz = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f32x4 z = *(const f32x4*)(&sZ[4][16 * r + 4 * L.g]);
#pragma unroll
            for (int b = 0; b < 3; ++b)
                if (b < L.w) z = z_then(z, block_bits(m, b), *(const f32x4*)(&sZ[b][16 * r + 4 * L.g]));
#pragma unroll
            for (int s = 0; s < 4; ++s) qz = __builtin_fmaf(qr[r][s], z[s], qz);
        }
        den = sum_g(den + (cont ? qz : 0.0f));
        // one reciprocal per row (correctly rounded) and a product per output
        if (L.g == 0) sDen[16 * L.w + L.c] = 1.0f / den;

        // ---- the four blocks in order against the wavefront's 16 columns
        f32x4 o[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t mb = block_bits(m, b);
            Frag kc;
            lds_rf(qr, sQ, 16 * b, L);
            lds_cf(kc, sK, 16 * b, L);
            o[b] = mul_state(st, qr);
            if (mb) o[b] = select4((mb & ((2u << L.c) - 1u)) == 0u, o[b]);
            o[b] = mul_slice_kept(vs[b], sA[b][L.lane], bit_range(first_of(mb, L.c), L.c + 1), o[b], L);
            if (mb) {
                const uint32_t keep = bit_range(31 - __builtin_clz(mb), kBlk);
                select_rows(kc, keep, L);
                select_rows(vs[b], keep, L);
#pragma unroll
                for (int s = 0; s < 4; ++s) st[s] = zero4();
            }
            state_add(st, kc, vs[b]);
        }
        fetch_v(ch + 1);
        barrier_lds();
        const ChunkRows co = chunk_rows(p.out, t0, p.T, p.H, h);
#pragma unroll
        for (int b = 0; b < 4; ++b) co.store_nt(16 * b + L.c, 16 * L.w + 4 * L.g, o[b] * sDen[16 * b + L.c]);
        if (L.w == 3) {                                           // z before the next chunk
            float z = sZ[4][L.lane];
#pragma unroll
            for (int b = 0; b < 4; ++b) z = block_bits(m, b) ? sZ[b][L.lane] : z + sZ[b][L.lane];
            sZ[4][L.lane] = z;
        }
    }

    if (want_idx && L.w == 1) {
        uint32_t count = seg == 0 ? 0u : count_lookback(p.cnt, seg - 1, 1, p.timeout);
        for (int ch = 0; ch < nch; ++ch) {
            const int64_t t0 = seg0 + (int64_t)ch * kChunk;
            const int64_t t = t0 + L.lane;
            const uint64_t mk = __ballot(t < p.T && (t == 0 || fetch_flag(p.start, t0, p.T) != 0u));
            if (t < p.T) p.idx[t] = (int32_t)(count + __builtin_popcountll(mk & ((2ull << L.lane) - 1ull))) - 1;
            count += (uint32_t)__builtin_popcountll(mk);
        }
        if (L.lane == 0 && seg > 0) publish64(p.cnt + seg, kCountIncl | count);
    }
}

// ------------------------------------------------------------------ launch

hipError_t linattn_summary_launch(const LinSummaryArgs& a, int64_t nseg, hipStream_t s) {
    hipLaunchKernelGGL(linattn_summary_kernel, dim3((unsigned)nseg, (unsigned)a.H), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <bool REV>
static void scan_launch(const LinScanArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)(a.width / (4 * kScanCols))), block(256);
    // the fewest rows per thread that take all segments at once
    if (a.n <= 2 * kScanGroups) hipLaunchKernelGGL((state_scan_kernel<2, REV>), grid, block, 0, s, a);
    else if (a.n <= 4 * kScanGroups) hipLaunchKernelGGL((state_scan_kernel<4, REV>), grid, block, 0, s, a);
    else if (a.n <= 8 * kScanGroups) hipLaunchKernelGGL((state_scan_kernel<8, REV>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((state_scan_kernel<kLinScanMaxRows, REV>), grid, block, 0, s, a);
}

hipError_t linattn_scan_launch(bool rev, const LinScanArgs& a, hipStream_t s) {
    if (rev) scan_launch<true>(a, s);
    else scan_launch<false>(a, s);
    return hipGetLastError();
}

hipError_t linattn_output_launch(const LinOutputArgs& a, int64_t nseg, hipStream_t s) {
    const dim3 grid((unsigned)nseg, (unsigned)a.H), block(256);
    if (nseg <= kLinDirectSegs) hipLaunchKernelGGL(linattn_output_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(linattn_output_kernel<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace memoroid
