// linattn_bwd.hip -- gradient of the linear-transformer memoroid readout
// (App. G.1) over a tape with resets, in segments of 64-row chunks like the
// forward pass, for gfx950.
//
// With Q = phi(q), K = phi(k), the forward states (S, z) and g = dL/dout:
//   dnum_i = g_i / den_i,  dden_i = -(g_i . out_i) / den_i,
//   dP     = (dnum V^T + dden 1^T) masked to the forward pattern M (j <= i,
//            j >= first(i): row i's episode inside the block),
//   dQ     = dP K + [row i's episode began earlier] (S dnum_i + dden_i z),
//   dK     = dP^T Q + [row j's episode runs past the block] (U v_j + w),
//   dV     = (A (.) M)^T dnum + [same] U^T K_j,
// where (S, z) is the state before the block and (U, w) the reverse state after
// it: sums of Q_t dnum_t^T and dden_t Q_t over the later steps of the episode.
//
// Kernels: the forward summary and state scan (linattn.hip) give the states
// before each segment; the dq kernel walks each segment forwards with (S, z)
// in registers, forming den (kept as 1 / den with dden, one float each per
// row), dnum, dq, and the segment's reverse summary (Q dnum^T and dden Q over
// its rows before its first begin step); the reverse state scan (cut at every
// segment that holds a begin step) gives the states after each segment; the
// dk/dv kernel walks each segment backwards.
#include "linattn_common.hpp"

namespace memoroid {

// ------------------------------------------------------------------- dq
// LDS: phi(Q), phi(K), V and dnum of the chunk (70 KB, two workgroups per CU).
// T = 32768, 4 heads: 62 us in a trace (64 over several sets of buffers), 227
// MFMAs a chunk and wavefront (24 us, matrix cores 45 % busy, counted); a
// separate backward-summary kernel and a dq product beside dk and dv took 44 us
// and a good third of 110, over several sets of buffers too.
template <bool DIRECT>
__global__ __launch_bounds__(256, 2) void linattn_dq_kernel(LinBwdArgs p) {
    __shared__ __attribute__((aligned(16))) float sQ[kTileF], sK[kTileF], sV[kTileF], sD[kTileF];
    __shared__ f32x4 sP[4][64];                                   // each block's masked dP, as mul_rows returns it
    __shared__ __attribute__((aligned(16))) float sZ[5][kDim];    // column sums of each block; [4]: z before the chunk
    __shared__ float sDd[kChunk];                                 // dden of the chunk's rows
    const int64_t seg = blockIdx.x, h = blockIdx.y;
    const LinLane L;
    const int64_t seg0 = seg * p.chunks * kChunk;
    const int64_t left = (p.T - seg0 + kChunk - 1) / kChunk;
    const int nch = (int)(left < p.chunks ? left : p.chunks);

    Frag qreg, kreg, vreg, gr, orow;           // gr, orow: row fragments of block w
    uint32_t flag;
    auto fetch_qkv = [&](int ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const bool have = ch < nch;
        flag = fetch_flag(p.start, have ? t0 : 0, have ? p.T : 0);
        fetch_chunk(kreg, chunk_rows(p.k, t0, p.T, p.H, h, have), L);
        fetch_chunk(qreg, chunk_rows(p.q, t0, p.T, p.H, h, have), L);
        fetch_chunk(vreg, chunk_rows(p.v, t0, p.T, p.H, h, have), L);
    };
    auto fetch_go = [&](int ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const ChunkRows cg = chunk_rows(p.g, t0, p.T, p.H, h, ch < nch), co = chunk_rows(p.out, t0, p.T, p.H, h, ch < nch);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            gr[r] = cg.load(16 * L.w + L.c, 16 * r + 4 * L.g);
            orow[r] = co.load(16 * L.w + L.c, 16 * r + 4 * L.g);
        }
    };
    fetch_qkv(0);
    fetch_go(0);
    Frag st, us;                               // st[s][r] = S[16 w + c][16 r + 4 g + s], us the same of U
    float z_in = 0.0f;
    state_before<DIRECT, false>(
        p.states, p.R, seg, p.nseg, p.H, h,
        [&](Rsrc rs) {
            load_state_n(st, rs, L);
            z_in = state_z1(rs, L.lane);
        },
        [&](Rsrc rs) {
            Frag s;
            load_state_n(s, rs, L);
            z_in += state_z1(rs, L.lane);
            add_frag(st, s);
        });
    if (L.w == 0) sZ[4][L.lane] = z_in;
#pragma unroll
    for (int s = 0; s < 4; ++s) us[s] = zero4();
    float ws = 0.0f;                           // reverse summary of w, column 16 w + c, this lane's rows
    bool head = true;                          // no begin step in the segment so far

#pragma unroll 1
    for (int ch = 0; ch < nch; ++ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const uint64_t m = begin_bits(flag, t0, p.T);
        stage_chunk<true>(sK, kreg, L);
        stage_chunk<true>(sQ, qreg, L);
        stage_chunk<false>(sV, vreg, L);
        barrier_lds();
        fetch_qkv(ch + 1);

        // ---- block w alone: den, dnum, dden, dP
        const uint32_t mw = block_bits(m, L.w);
        const int first = first_of(mw, L.c);
        const bool cont = (mw & ((2u << L.c) - 1u)) == 0u;       // row c's episode began before the block
        Frag qr;
        float den = 0.0f;
        {
            Frag kr;
            lds_rf(kr, sK, 16 * L.w, L);
            lds_rf(qr, sQ, 16 * L.w, L);
            const f32x4 at = mul_rows(kr, qr);                    // phi(k_j) . phi(q_c), j = 4 g + r
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = 4 * L.g + r;
                den += j <= L.c && j >= first ? at[r] : 0.0f;
            }
            Frag kc;
            lds_cf(kc, sK, 16 * L.w, L);
            if (mw) select_rows(kc, bit_range(31 - __builtin_clz(mw), kBlk), L);
            const f32x4 zs = col_sums(kc, f32x4{1.0f, 1.0f, 1.0f, 1.0f});
            if (L.g == 0) *(f32x4*)(&sZ[L.w][L.cm]) = zs;
        }
        barrier_lds();
        {
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
            const float rden = 1.0f / den;
            const float dd = -sum_g(dot_frag(gr, orow)) * rden;
            Frag vr;
            lds_rf(vr, sV, 16 * L.w, L);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gr[r] *= rden;                                    // dnum
                *(f32x4*)(sD + (16 * L.w + L.c) * kLD + 16 * r + 4 * L.g) = gr[r];
            }
            f32x4 dp = mul_rows(vr, gr);                          // v_j . dnum_c
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = 4 * L.g + r;
                dp[r] = j <= L.c && j >= first ? dp[r] + dd : 0.0f;
            }
            sP[L.w][L.lane] = dp;
            if (L.g == 0) {
                const int64_t t = t0 + 16 * L.w + L.c;
                sDd[16 * L.w + L.c] = dd;
                if (t < p.T) {
                    p.rden[t * p.H + h] = rden;
                    p.dden[t * p.H + h] = dd;
                }
            }
        }
        barrier_lds();
        fetch_go(ch + 1);

        // ---- the four blocks in order against the wavefront's 16 columns kd
        f32x4 z = *(const f32x4*)(&sZ[4][16 * L.w + 4 * L.g]);
        const ChunkRows cq = chunk_rows(p.dq, t0, p.T, p.H, h);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t mb = block_bits(m, b);
            Frag x;
            lds_rf(x, sD, 16 * b, L);
            f32x4 ks = lds_slice(sK, 16 * b, L);
            f32x4 acc = mul_state(st, x);                         // S dnum_c
            const float dd = sDd[16 * b + L.c];
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = __builtin_fmaf(dd, z[r], acc[r]);
            if (mb) acc = select4((mb & ((2u << L.c) - 1u)) == 0u, acc);
            acc = mul_slice_kept(ks, sP[b][L.lane], bit_range(first_of(mb, L.c), L.c + 1), acc, L);
            const f32x4 qv = *(const f32x4*)(sQ + (16 * b + L.c) * kLD + 16 * L.w + 4 * L.g);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] *= phi_prime_of_phi(qv[r]);
            cq.store_nt(16 * b + L.c, 16 * L.w + 4 * L.g, acc);
            z = z_then(z, mb, *(const f32x4*)(&sZ[b][16 * L.w + 4 * L.g]));
            // the segment's rows before its first begin, for the reverse state
            if (head) {
                lds_cf(x, sD, 16 * b, L);
                f32x4 qs = lds_slice(sQ, 16 * b, L);
                f32x4 ds;
#pragma unroll
                for (int q = 0; q < 4; ++q) ds[q] = sDd[16 * b + 4 * L.g + q];
                if (mb) {
                    const uint32_t keep = bit_range(0, __builtin_ctz(mb));
                    select_rows(x, keep, L);
                    select_rows(qs, keep, L);
                    select_rows(ds, keep, L);
                    head = false;
                }
                state_add_once(us, x, qs);
                float wb = 0.0f;
#pragma unroll
                for (int q = 0; q < 4; ++q) wb = __builtin_fmaf(ds[q], qs[q], wb);
                ws += wb;
            }
            lds_cf(x, sV, 16 * b, L);
            if (mb) {
                const uint32_t keep = bit_range(31 - __builtin_clz(mb), kBlk);
                select_rows(x, keep, L);
                select_rows(ks, keep, L);
#pragma unroll
                for (int s = 0; s < 4; ++s) st[s] = zero4();
            }
            state_add_once(st, x, ks);
        }
        // every wavefront has read all of z before the chunk (it is past the
        // barrier above) but its own quarter, which it rewrites here
        if (L.c == 0) *(f32x4*)(&sZ[4][16 * L.w + 4 * L.g]) = z;
        barrier_lds();
    }
    float* const out = p.rstates + (seg * p.H + h) * kStateWords;
    store_state_n(out, us, L);
    ws = sum_g(ws);
    if (L.g == 0) out[kDim * kDim + 16 * L.w + L.c] = ws;
}

// --------------------------------------------------------------- dk and dv
// LDS: phi(Q), phi(K), V and dnum of the chunk (70 KB, two workgroups per CU).
// dk contracts U over its columns and dv over its rows, so U is kept in both
// register layouts (64 MFMAs a chunk and wavefront more than one copy would
// take).  T = 32768, 4 heads: 66 us in a trace (68 over several sets of
// buffers), 320 MFMAs a chunk and wavefront (34 us, matrix cores 59 % busy,
// counted).  Before block sums were formed apart, at 61 us a call: 54 us with
// every load served by the L2, 46 us with the MFMAs replaced by single FMAs.
template <bool DIRECT>
__global__ __launch_bounds__(256, 2) void linattn_dkv_kernel(LinBwdArgs p) {
    __shared__ __attribute__((aligned(16))) float sQ[kTileF], sK[kTileF], sV[kTileF], sD[kTileF];
    __shared__ f32x4 sP[4][64], sA[4][64];                        // each block's masked dP and A
    __shared__ __attribute__((aligned(16))) float sW[4][kDim];    // sums of dden Q over each block's head
    const int64_t seg = blockIdx.x, h = blockIdx.y;
    const LinLane L;
    const int64_t seg0 = seg * p.chunks * kChunk;
    const int64_t left = (p.T - seg0 + kChunk - 1) / kChunk;
    const int nch = (int)(left < p.chunks ? left : p.chunks);

    Frag qreg, kreg, vreg, greg;
    f32x4 rd, dd;                              // 1 / den of the staged rows, dden of block w's rows 4 g + r
    uint32_t flag;
    auto fetch = [&](int ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const bool have = ch >= 0;
        flag = fetch_flag(p.start, have ? t0 : 0, have ? p.T : 0);
        const ChunkRows cr = row_scalars(p.rden, t0, p.T, p.H, h, have), cd = row_scalars(p.dden, t0, p.T, p.H, h, have);
#pragma unroll
        for (int u = 0; u < 4; ++u) rd[u] = cr.load1(16 * u + (L.tid >> 4), 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) dd[r] = cd.load1(16 * L.w + 4 * L.g + r, 0);
        fetch_chunk(greg, chunk_rows(p.g, t0, p.T, p.H, h, have), L);
        fetch_chunk(vreg, chunk_rows(p.v, t0, p.T, p.H, h, have), L);
        fetch_chunk(qreg, chunk_rows(p.q, t0, p.T, p.H, h, have), L);
        fetch_chunk(kreg, chunk_rows(p.k, t0, p.T, p.H, h, have), L);
    };
    fetch(nch - 1);
    Frag uk, uv;                               // uk[s][r] = U[16 w + c][16 r + 4 g + s], uv[s][r] = U[16 r + 4 g + s][16 w + c]
    f32x4 wz = zero4();
    const int wat = 16 * L.w + 4 * L.g;
    state_before<DIRECT, true>(
        p.rstates, p.R, seg, p.nseg, p.H, h,
        [&](Rsrc rs) {
            load_state_n(uk, rs, L);
            load_state_kd(uv, rs, L);
            wz = state_z4(rs, wat);
        },
        [&](Rsrc rs) {
            Frag sk, sv;
            load_state_n(sk, rs, L);
            load_state_kd(sv, rs, L);
            wz += state_z4(rs, wat);
            add_frag(uk, sk);
            add_frag(uv, sv);
        });

#pragma unroll 1
    for (int ch = nch - 1; ch >= 0; --ch) {
        const int64_t t0 = seg0 + (int64_t)ch * kChunk;
        const uint64_t m = begin_bits(flag, t0, p.T);
#pragma unroll
        for (int u = 0; u < 4; ++u) greg[u] *= rd[u];             // dnum
        stage_chunk<false>(sD, greg, L);
        stage_chunk<false>(sV, vreg, L);
        stage_chunk<true>(sQ, qreg, L);
        stage_chunk<true>(sK, kreg, L);
        const f32x4 ddw = dd;
        barrier_lds();
        fetch(ch - 1);

        // ---- block w alone: dP and A (row i = 4 g + r against row c), and the
        // sums of dden Q over its rows before its first begin
        {
            const uint32_t mw = block_bits(m, L.w);
            const int end = end_of(mw, L.c);
            Frag x, y;
            lds_rf(x, sD, 16 * L.w, L);
            lds_rf(y, sV, 16 * L.w, L);
            f32x4 a = mul_rows(x, y);                             // dnum_i . v_c
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * L.g + r;
                a[r] = i >= L.c && i < end ? a[r] + ddw[r] : 0.0f;
            }
            sP[L.w][L.lane] = a;
            lds_rf(x, sQ, 16 * L.w, L);
            lds_rf(y, sK, 16 * L.w, L);
            a = mul_rows(x, y);                                   // phi(q_i) . phi(k_c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * L.g + r;
                a[r] = i >= L.c && i < end ? a[r] : 0.0f;
            }
            sA[L.w][L.lane] = a;
            lds_cf(x, sQ, 16 * L.w, L);
            f32x4 dw = ddw;
            if (mw) {
                const uint32_t keep = bit_range(0, __builtin_ctz(mw));
                select_rows(x, keep, L);
                select_rows(dw, keep, L);
            }
            const f32x4 wsum = col_sums(x, dw);
            if (L.g == 0) *(f32x4*)(&sW[L.w][L.cm]) = wsum;
        }
        barrier_lds();

        // ---- the four blocks from the last back, against the wavefront's 16
        // columns (kd of dk, n of dv)
        const ChunkRows ck = chunk_rows(p.dk, t0, p.T, p.H, h), cv = chunk_rows(p.dv, t0, p.T, p.H, h);
#pragma unroll
        for (int b = 3; b >= 0; --b) {
            const uint32_t mb = block_bits(m, b);
            const int end = end_of(mb, L.c);
            const uint32_t keep = bit_range(L.c, end);
            Frag x;
            f32x4 qs = lds_slice(sQ, 16 * b, L), ds = lds_slice(sD, 16 * b, L);
            lds_rf(x, sV, 16 * b, L);
            f32x4 acc = mul_state(uk, x) + wz;                    // U v_c + w
            if (mb) acc = select4(end == kBlk, acc);              // row c's episode runs past the block
            acc = mul_slice_kept(qs, sP[b][L.lane], keep, acc, L);
            const f32x4 kv = *(const f32x4*)(sK + (16 * b + L.c) * kLD + 16 * L.w + 4 * L.g);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] *= phi_prime_of_phi(kv[r]);
            ck.store_nt(16 * b + L.c, 16 * L.w + 4 * L.g, acc);
            lds_rf(x, sK, 16 * b, L);
            acc = mul_state(uv, x);                               // U^T phi(k_c)
            if (mb) acc = select4(end == kBlk, acc);
            acc = mul_slice_kept(ds, sA[b][L.lane], keep, acc, L);
            cv.store_nt(16 * b + L.c, 16 * L.w + 4 * L.g, acc);
            // the state before the block
            wz = z_then(wz, mb, *(const f32x4*)(&sW[b][16 * L.w + 4 * L.g]));
            Frag y;
            lds_cf(x, sD, 16 * b, L);
            lds_cf(y, sQ, 16 * b, L);
            if (mb) {
                const uint32_t hd = bit_range(0, __builtin_ctz(mb));
                select_rows(x, hd, L);
                select_rows(y, hd, L);
                select_rows(qs, hd, L);
                select_rows(ds, hd, L);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    uk[s] = zero4();
                    uv[s] = zero4();
                }
            }
            state_add_once(uk, x, qs);
            state_add(uv, y, ds);
        }
        barrier_lds();
    }
}

hipError_t linattn_dq_launch(const LinBwdArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)a.nseg, (unsigned)a.H), block(256);
    if (a.nseg <= kLinDirectSegs) hipLaunchKernelGGL(linattn_dq_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(linattn_dq_kernel<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t linattn_dkv_launch(const LinBwdArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)a.nseg, (unsigned)a.H), block(256);
    if (a.nseg <= kLinDirectSegs) hipLaunchKernelGGL(linattn_dkv_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(linattn_dkv_kernel<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace memoroid
