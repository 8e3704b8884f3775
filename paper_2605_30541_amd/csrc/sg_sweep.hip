// Column-sweep time blocking of the forward step (SubsurfaceGen, arXiv
// 2605.30541: eqs. "acoustic_2d", "cerjan_pde", "free_surface"; App. E.3), for
// launches with many workgroups (many shots):
//   p^{n+1} = W L p^n + (2a (p^n - p^{n-1}) + p^{n-1}) + W S^n
// on every padded cell, the same expression and operation order as the tiled
// kernel (sg_kernels.hip), so both give the same bits.
//
// A workgroup owns one strip of 64 NW columns of one shot (its output columns
// plus a halo of 4 tb on each side) and walks the whole height of the padded
// grid once per launch, advancing TB levels in a skewed pipeline: at step j it
// takes level n at row j from memory and computes level n+s at row j - 4s for
// s = 1..TB.  Level n+s at row R needs level n+s-1 at rows R-4..R+4, which
// the previous level finished at this step or before, so nothing in z is
// recomputed; only the x halo is.  Each level keeps its last 9 rows (the
// stencil's reach) in registers -- z neighbours come from there -- and in a
// 9-row LDS ring for the x neighbours of the next level.  The step loop is
// unrolled by 9 so queue and ring slots are compile-time constants.
//
// Boundaries without branches: loads are clamped into the 4-cell zero guard
// ring of the stored fields, so rows and columns outside the padded grid read
// p = 0 with W = 2a = 0 and every value computed there is exactly 0; the
// pinned free-surface row has W = 2a = 0 too and stays 0.  Under a free top
// the ghost rows -1..-4 of every level hold minus rows 1..4 (odd mirror):
// when a level produces row R in 1..4 it writes -p into the register slot of
// row -R, before any row that reads it is computed.
//
// Bound: vector issue (71 % of the cycles a CU has work, 256-column strips,
// time block 5; 26 to 28 vector instructions per lane and update in the plain
// steps, 20 of them the Laplacian), then the share of a strip's lanes that is
// halo.  8 uneven slices x 32 shots x 400 updates: 114.1 ms with one form for
// all steps (best at time block 4, 320-row segments), 87.5 ms with runs of plain
// steps (time block 5, equal segments of up to 160 rows).
#include "sg_internal.h"

#include <type_traits>

namespace sg {

namespace {

constexpr int kQ = 9;   // rows of a level kept: R-4..R+4

template <class T>
__device__ __forceinline__ T gld(const T *p)
{
    return *(const __attribute__((address_space(1))) T *)p;
}
template <class T>
__device__ __forceinline__ T gld_at(const T *base, uint32_t byte_off)
{
    return gld((const T *)((const char *)base + byte_off));
}
__device__ __forceinline__ void gst_at(float *base, uint32_t byte_off, float v)
{
    *(__attribute__((address_space(1))) float *)((char *)base + byte_off) = v;
}

// Register / ring slot of a row, row = j + d at a step j with j mod 9 = PH.
constexpr int slot(int d) { return ((d % kQ) + kQ) % kQ; }

__device__ inline int xcd_block(int b, int nblocks)
{
    const int per = nblocks >> 3;
    if (b >= per * 8) return b;
    return (b & 7) * per + (b >> 3);
}

// RECOMP (the forward recompute of the gradient): also stores, for every level
// n+q-1 advanced, the second time difference D = (p^{n+q} - p^{n+q-1}) -
// (p^{n+q-1} - p^{n+q-2}) of the output cells in ring slot n+q-1 - t.ring_lo
// (streaming stores: read back only by the adjoint after the segment).
template <int NW, int TB, bool RECOMP>
__device__ __forceinline__ void sweep_body(const SliceDesc &s, const TileArgs &t, int b, float *lds)
{
    constexpr int EX = 64 * NW, LW = EX + 2 * kHalo, NTHR = 64 * NW, RING = kQ * LW;
    // block b: (shot, segment, strip); a segment is the output rows
    // [zs0, zs1) of the strip (t.tz rows; one segment = the whole height)
    const int tiles = t.ntx * t.ntz;
    const int shot = b / tiles;
    const int tile = b - shot * tiles;
    const int seg = tile / t.ntx;
    const int strip = tile - seg * t.ntx;
    const int zs0 = seg * t.tz, zs1 = min(zs0 + t.tz, s.Nz);
    const int ox = strip * t.tx, ox_end = min(ox + t.tx, s.Nx), ex0 = ox - kHalo * t.tb;
    const int lx = (int)threadIdx.x;
    const int X = ex0 + lx;
    const bool xout = X >= ox && X < ox_end;
    // clamped into the guard columns (zeros): no test on columns outside the grid
    const int Xc = min(max(X, -kGuard), s.Nx + kGuard - 1);
    const uint32_t xo4 = (uint32_t)(Xc + kGuard) * 4u;
    const int pitch = s.pitch, Nz = s.Nz;
    auto rowb = [&](int R) -> uint32_t {                    // clamped into the guard rows (zeros)
        R = min(max(R, -kGuard), Nz + kGuard - 1);
        return (uint32_t)((R + kGuard) * pitch) * 4u;
    };
    const float *in_prev = t.in + (int64_t)shot * t.in_shot;
    const float *in_cur = in_prev + s.frame;
    float *out_prev = t.out + (int64_t)shot * t.out_shot;
    float *out_cur = out_prev + s.frame;
    const bool free_top = s.free_top != 0;

    // rows holding source nodes of this shot in this strip's columns (srow_lo
    // and srow_hi, one below the other or the same) and this lane's node weight
    // on each of them; the wavelet samples are read only there (level n+s takes
    // w(t_{n+s-1})).  Strips beside the source have none, and run plain steps.
    const float *wshot = s.wavelet + (int64_t)shot * s.wavelet_stride + t.n;
    int srow_lo = 1 << 30, srow_hi = -(1 << 30);
    float sw_lo = 0.f, sw_hi = 0.f;
    {
        int iz[kNodes], ixn[kNodes];
        float wn[kNodes];
#pragma unroll
        for (int k = 0; k < kNodes; ++k) {
            iz[k] = gld(s.src_iz + shot * kNodes + k);
            ixn[k] = gld(s.src_ix + shot * kNodes + k);
            wn[k] = gld(s.src_w + shot * kNodes + k);
            if (ixn[k] < ex0 || ixn[k] >= ex0 + EX) wn[k] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < kNodes; ++k)
            if (wn[k] != 0.f) {
                srow_lo = min(srow_lo, iz[k]);
                srow_hi = max(srow_hi, iz[k]);
            }
        // (the four nodes of a point are four cells: at most one per row and lane)
#pragma unroll
        for (int k = 0; k < kNodes; ++k)
            if (wn[k] != 0.f && ixn[k] == X) {
                if (iz[k] == srow_lo) sw_lo = wn[k];
                if (iz[k] == srow_hi) sw_hi = wn[k];
            }
        srow_lo = __builtin_amdgcn_readfirstlane(srow_lo);
        srow_hi = __builtin_amdgcn_readfirstlane(srow_hi);
    }
    // receivers of this strip (entries sorted by base row); levels n..n+TB-1 due
    int rbeg = 0, rend = 0, rrow_lo = 1 << 30, rrow_hi = -(1 << 30);
    unsigned due = 0;
    if (!RECOMP && s.gathers) {   // (a recompute records nothing)
        rbeg = gld(s.tile_rec + tile);
        rend = gld(s.tile_rec + tile + 1);
        if (rend > rbeg) {
            rrow_lo = gld(&s.rec_list[rbeg].lds) / LW;
            rrow_hi = gld(&s.rec_list[rend - 1].lds) / LW;
        }
#pragma unroll
        for (int q = 0; q < TB; ++q)
            if ((t.n + q) % s.rec_every == 0 && q < t.nsteps) due |= 1u << q;
    }
    // steps at which some due level records a receiver row (one range test per step)
    const int rec_j0 = __builtin_amdgcn_readfirstlane(due && rend > rbeg ? rrow_lo + 6 : 1 << 30);
    const int rec_j1 =
        __builtin_amdgcn_readfirstlane(due && rend > rbeg ? rrow_hi + 4 * (TB - 1) + 6 : -(1 << 30));

    float Q[TB][kQ];
#pragma unroll
    for (int a = 0; a < TB; ++a)
#pragma unroll
        for (int c = 0; c < kQ; ++c) Q[a][c] = 0.f;
    // this lane's column in ring row 0 of level 0, as a byte address
    const int lane_b = (lx + kHalo) * 4;
    float *const my = lds + lx + kHalo;
    // zero the rings (pad columns included: read only by discarded halo cells)
    for (int q = threadIdx.x; q < TB * RING; q += NTHR) lds[q] = 0.f;

    // Loads of the two input levels run two steps ahead of their use: step j
    // takes level n at row j and level n-1 at row j-4 from prefetch slot j mod 3
    // (3 divides the unroll of 9, so slots are compile-time too) and issues the
    // loads of step j+2 into slot (j+2) mod 3.  W and 2a of the rows j-4q go the
    // same way at time blocks up to 3; beyond, where 16 more registers would
    // spill, they are loaded one step ahead, level n+q's for step j+1 into the
    // register its step j has just used (mostly from L2: every level reads each
    // row in turn).  Time block 3 with one step ahead: 5 % slower.
    constexpr int kPf = 3, kPw = TB <= 3 ? 3 : 1, kAhead = TB <= 3 ? 2 : 1;
    float pc[kPf], pp[kPf], pw[kPw][TB], pa[kPw][TB];
    auto issue = [&](const int slotp, const int jj) {
        pc[slotp] = gld_at(in_cur, rowb(jj) + xo4);
        pp[slotp] = gld_at(in_prev, rowb(jj - 4) + xo4);
    };
    auto issue_coef = [&](const int slotw, const int q, const int jj) {   // q = 1 .. TB
        const uint32_t o = rowb(jj - 4 * q) + xo4;
        pw[slotw][q - 1] = gld_at(s.W, o);
        pa[slotw][q - 1] = gld_at(s.A2, o);
    };
    // first step: the top segment starts at row -9 (every row above 0 is a
    // guard or ghost row); a lower one TB levels of 4 rows, plus the 4 rows
    // level n+1 reads above, before its first output row, on a multiple of 9
    // (the unrolled loop's phase 0): rows computed before then are not exact,
    // and no output row reads them
    const int jf = zs0 - 4 * TB - kHalo;
    const int j0 = zs0 == 0 ? -kQ : jf - (jf % kQ + kQ) % kQ;
    pc[2] = pp[2] = 0.f;   // (filled at the first step)
#pragma unroll
    for (int q = 1; q <= TB; ++q) {
#pragma unroll
        for (int u = 0; u < kPw; ++u) {
            if (u < kAhead)
                issue_coef(u, q, j0 + u);
            else
                pw[u][q - 1] = pa[u][q - 1] = 0.f;   // (filled at the first step)
        }
    }
    issue(0, j0);
    issue(1, j0 + 1);

    // The plain steps: rows past the free top's ghost rows, no source row and no
    // receiver sample among them or below them in the strip's segment.  What the
    // others test for (mirror, sources, receivers, rows above the grid, with the
    // scalar registers that spills) is a third of their instructions, so a group
    // of kQ plain steps runs in a form without it, and on strips and rows where
    // every cell has a = 1 (UNIT) without loading 2a.  With sources and receivers
    // near the surface nearly all steps are plain; a deep source keeps its own
    // strip's segment in the general form down to it, deep receivers theirs.  16
    // shots x 100 updates of 620 x 1001 cells (256-column strips, 160-row segments,
    // time block 5), in the general form throughout and now: all at the surface
    // 3.64 and 2.34 ms, sources at 92 % of the depth 3.76 and 2.72, receivers there
    // 3.76 and 2.87, receivers down a vertical line 8.62 and 5.07.
    // byte offset of a row past the ghost rows; below the grid that of the last guard row
    auto rowp = [&](int R) -> uint32_t { return (uint32_t)((min(R, Nz + kGuard - 1) + kGuard) * pitch) * 4u + xo4; };
    auto plain_step = [&](auto ph, auto unit, const int j) {
        constexpr int PH = decltype(ph)::value;
        constexpr bool UNIT = decltype(unit)::value;
        constexpr int PS = PH % kPf;
        pc[(PH + 2) % kPf] = gld_at(in_cur, rowp(j + 2));
        pp[(PH + 2) % kPf] = gld_at(in_prev, rowp(j - 2));
        if (PH % 3 == 0) __syncthreads();
        const float cin = pc[PS];
        Q[0][slot(PH)] = cin;
        my[slot(PH) * LW] = cin;
        float vlast = 0.f;
#pragma unroll
        for (int q = 1; q <= TB; ++q) {
            const float(&P)[kQ] = Q[q - 1];
            const float c = P[slot(PH - 4 * q)];
            int xa = lane_b + ((q - 1) * RING + slot(PH - 4 * q) * LW - kHalo) * 4;   // column x - 4
            asm volatile("" : "+v"(xa));
            const float *xr = (const float *)((const char *)lds + xa);
            const float c4 = -4.f * c;
            float lap = 0.f;
#pragma unroll
            for (int m = 1; m <= kHalo; ++m) {
                const float zs = P[slot(PH - 4 * q + m)] + P[slot(PH - 4 * q - m)];
                lap = fmaf(s.cz[m], (zs + (xr[kHalo + m] + xr[kHalo - m])) + c4, lap);
            }
            const float old = q == 1 ? pp[PS] : Q[q - 2][slot(PH - 4 * q)];
            const float v = fmaf(pw[PH % kPw][q - 1], lap, fmaf(UNIT ? 2.f : pa[PH % kPw][q - 1], c - old, old));
            {
                const uint32_t o = rowp(j + kAhead - 4 * q);
                pw[(PH + kAhead) % kPw][q - 1] = gld_at(s.W, o);
                if (!UNIT) pa[(PH + kAhead) % kPw][q - 1] = gld_at(s.A2, o);
            }
            if (RECOMP && xout && j - 4 * q >= zs0 && j - 4 * q < zs1) {
                float *rl = t.ring + (int64_t)shot * t.ring_shot + (int64_t)(t.n + q - 1 - t.ring_lo) * s.frame;
                __builtin_nontemporal_store((v - c) - (c - old),
                                            (__attribute__((address_space(1))) float *)((char *)rl +
                                                (uint32_t)((j - 4 * q + kGuard) * pitch) * 4u + xo4));
            }
            if (q < TB) {
                Q[q][slot(PH - 4 * q)] = v;
                my[q * RING + slot(PH - 4 * q) * LW] = v;
            } else {
                vlast = v;
            }
        }
        if (xout && j - 4 * TB >= zs0 && j - 4 * TB < zs1) {
            const uint32_t o = (uint32_t)((j - 4 * TB + kGuard) * pitch) * 4u + xo4;
            gst_at(out_cur, o, vlast);
            gst_at(out_prev, o, Q[TB - 1][slot(PH - 4 * TB)]);
        }
    };

    auto step = [&](auto ph, const int j) {
        constexpr int PH = decltype(ph)::value;
        constexpr int PS = PH % kPf;
        // loads of step j+2 (slot (PH+2) mod 3 was last read at step j-1)
        issue((PH + 2) % kPf, j + 2);
        // A level's ring row written at step j is read by other waves at step
        // j+4 (x neighbours of the next level) and rows written at steps j-6,
        // j-5 by the receivers; the slot it overwrites was last read at step
        // j-5.  A barrier every third step orders both.
        if (PH % 3 == 0) __syncthreads();
        // level n, row j
        const float cin = pc[PS];
        Q[0][slot(PH)] = cin;
        my[slot(PH) * LW] = cin;
        if (free_top && j >= 1 && j <= kHalo) Q[0][slot(-PH)] = -cin;
        // receivers of levels n..n+TB-1 at base row j - 4q - 6: an entry's row
        // tells its level, so each is looked at once a step and not once for
        // every level (receivers down a vertical line, strips of the whole height,
        // time block 5: 47.9 -> 22.3 ms).  A loop, not unrolled: it touches no
        // register queue, and copies of it in every phase and level took registers
        // from the plain steps.
        if (!RECOMP && j >= rec_j0 && j <= rec_j1) {
            bool any = false;
#pragma unroll
            for (int q = 0; q < TB; ++q) {
                const int Rb = j - 4 * q - 6;
                any |= ((due >> q) & 1u) && Rb >= rrow_lo && Rb <= rrow_hi;
            }
            if (any) {
#pragma unroll 1
                for (int e = rbeg + (int)threadIdx.x; e < rend; e += NTHR) {
                    const int code = gld(&s.rec_list[e].lds), Rb = code / LW, c = code - Rb * LW;
                    const int d = j - 6 - Rb, q = d >> 2;
                    if (d < 0 || (d & 3) || q >= TB || !((due >> q) & 1u)) continue;
                    const int s0 = (PH + 8 * kQ - 4 * q - 6) % kQ, s1 = s0 + 1 == kQ ? 0 : s0 + 1;
                    const float *L0 = lds + q * RING + s0 * LW;
                    const float *L1 = lds + q * RING + s1 * LW;
                    float *row = s.gathers + ((int64_t)shot * s.nrow + (t.n + q) / s.rec_every) * s.nrec;
                    const float w0 = gld(&s.rec_list[e].w[0]), w1 = gld(&s.rec_list[e].w[1]);
                    const float w2 = gld(&s.rec_list[e].w[2]), w3 = gld(&s.rec_list[e].w[3]);
                    row[gld(&s.rec_list[e].r)] = w0 * L0[c] + w1 * L0[c + 1] + w2 * L1[c] + w3 * L1[c + 1];
                }
            }
        }
        // levels n+1 .. n+TB at rows j-4 .. j-4TB
        float vlast = 0.f;
#pragma unroll
        for (int q = 1; q <= TB; ++q) {
            const int R = j - 4 * q;
            const float(&P)[kQ] = Q[q - 1];
            const float c = P[slot(PH - 4 * q)];
            // x neighbours of level q-1 at row R: one address register per
            // read group (the empty asm keeps the compiler from folding the
            // ring offset into every read, which costs an add per pair)
            int xa = lane_b + ((q - 1) * RING + slot(PH - 4 * q) * LW - kHalo) * 4;   // column x - 4
            asm volatile("" : "+v"(xa));
            const float *xr = (const float *)((const char *)lds + xa);
            const float c4 = -4.f * c;
            float lap = 0.f;
#pragma unroll
            for (int m = 1; m <= kHalo; ++m) {
                const float zs = P[slot(PH - 4 * q + m)] + P[slot(PH - 4 * q - m)];
                lap = fmaf(s.cz[m], (zs + (xr[kHalo + m] + xr[kHalo - m])) + c4, lap);
            }
            const float old = q == 1 ? pp[PS] : Q[q - 2][slot(PH - 4 * q)];
            const float Wq = pw[PH % kPw][q - 1];
            float v = fmaf(Wq, lap, fmaf(pa[PH % kPw][q - 1], c - old, old));
            issue_coef((PH + kAhead) % kPw, q, j + kAhead);
            if (R == srow_lo || R == srow_hi) {
                const float wk = R == srow_lo ? sw_lo : sw_hi;
                if (wk != 0.f) v = fmaf(Wq, wk * gld(wshot + (q - 1)), v);
            }
            if (RECOMP && R >= zs0 && R < zs1 && xout) {
                float *rl = t.ring + (int64_t)shot * t.ring_shot + (int64_t)(t.n + q - 1 - t.ring_lo) * s.frame;
                __builtin_nontemporal_store((v - c) - (c - old),
                                            (__attribute__((address_space(1))) float *)((char *)rl +
                                                (uint32_t)((R + kGuard) * pitch) * 4u + xo4));
            }
            if (q < TB) {
                Q[q][slot(PH - 4 * q)] = v;
                my[q * RING + slot(PH - 4 * q) * LW] = v;
                if (free_top && R >= 1 && R <= kHalo) Q[q][slot(4 * q - PH)] = -v;
            } else {
                vlast = v;
            }
        }
        // output: levels n+TB and n+TB-1 at row j - 4TB
        const int R = j - 4 * TB;
        if (R >= zs0 && R < zs1 && xout) {
            const uint32_t o = (uint32_t)((R + kGuard) * pitch) * 4u + xo4;
            gst_at(out_cur, o, vlast);
            gst_at(out_prev, o, Q[TB - 1][slot(PH - 4 * TB)]);
        }
    };

    // steps j0 .. j1-1: guard rows outside [-4, Nz+4) read as the clamped
    // guard row; the last step computes level n+TB at row zs1-1, or later the
    // last receiver sample (a receiver on the segment's last two rows is read
    // 6 steps after its rows of level n+TB-1 are computed); the rings were
    // zeroed before the first step's barrier
    const int nsteps = max(zs1 + 4 * TB, rec_j1 + 1) - j0;
    const int j1 = j0 + (nsteps + kQ - 1) / kQ * kQ;
    // Three runs of groups, one after the other (each keeps its registers from
    // group to group; with a choice per group they were spilled): the steps up
    // to the last source row or receiver sample, or to the first row clear of
    // the ghost rows; the plain ones whose rows j - 4 TB .. j + 4 and columns
    // all have a = 1; the other plain ones, down to the guard rows.
    // (a source below the segment's last step is no source of the segment)
    const int jsrc = srow_lo < j1 - 4 ? srow_hi + 4 * TB : -(1 << 30);
    const int jp0 = max(4 * TB + kHalo + 1, max(jsrc, rec_j1) + 1);
    const bool unit_x = ex0 >= s.unit_x0 && ex0 + EX <= s.unit_x1;
    const int ju0 = max(jp0, s.unit_z0 + 4 * TB), ju1 = min(s.unit_z1 - (kQ - 1) + kHalo, Nz + kGuard - kQ - 1);
    auto group = [&](auto unit, const int j) {
        plain_step(std::integral_constant<int, 0>{}, unit, j);
        plain_step(std::integral_constant<int, 1>{}, unit, j + 1);
        plain_step(std::integral_constant<int, 2>{}, unit, j + 2);
        plain_step(std::integral_constant<int, 3>{}, unit, j + 3);
        plain_step(std::integral_constant<int, 4>{}, unit, j + 4);
        plain_step(std::integral_constant<int, 5>{}, unit, j + 5);
        plain_step(std::integral_constant<int, 6>{}, unit, j + 6);
        plain_step(std::integral_constant<int, 7>{}, unit, j + 7);
        plain_step(std::integral_constant<int, 8>{}, unit, j + 8);
    };
    int j = j0;
    for (; j < j1 && (j < jp0 || (unit_x && j < ju0)); j += kQ) {
        step(std::integral_constant<int, 0>{}, j);
        step(std::integral_constant<int, 1>{}, j + 1);
        step(std::integral_constant<int, 2>{}, j + 2);
        step(std::integral_constant<int, 3>{}, j + 3);
        step(std::integral_constant<int, 4>{}, j + 4);
        step(std::integral_constant<int, 5>{}, j + 5);
        step(std::integral_constant<int, 6>{}, j + 6);
        step(std::integral_constant<int, 7>{}, j + 7);
        step(std::integral_constant<int, 8>{}, j + 8);
    }
    if (unit_x && j < j1 && j < ju1) {
        for (; j < j1 && j < ju1; j += kQ) group(std::true_type{}, j);
        // 2a of the next kAhead steps, which these groups left out
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int q = 0; q < TB; ++q) pa[u][q] = gld_at(s.A2, rowb(j + u - 4 * (q + 1)) + xo4);
    }
    for (; j < j1; j += kQ) group(std::false_type{}, j);
}

#define SG_SWEEP_OCCUPANCY __attribute__((amdgpu_waves_per_eu(TB <= 4 ? 4 : (TB == 5 ? 3 : 2))))
template <int NW, int TB, bool RECOMP>
__global__ void __launch_bounds__(64 * NW) SG_SWEEP_OCCUPANCY k_sweep(SliceDesc s, TileArgs t)
{
    __shared__ float lds[TB * kQ * (64 * NW + 2 * kHalo)];
    sweep_body<NW, TB, RECOMP>(s, t, xcd_block(blockIdx.x, gridDim.x), lds);
}

template <int NW, int TB, bool RECOMP>
__global__ void __launch_bounds__(64 * NW) SG_SWEEP_OCCUPANCY k_sweep_batch(const BatchItem *__restrict__ items, int nitems, int n,
                                                                             LevelPair lv, int ring_lo, bool deal)
{
    __shared__ float lds[TB * kQ * (64 * NW + 2 * kHalo)];
    // Each XCD takes an eighth of the launch's tiles in order, or (`deal`) an
    // eighth of every item's.  The first gives an XCD one or two items, whose
    // segments may be higher than the others': eight slices of 459 to 629 rows
    // (153 to 210 a segment) left the shorter ones' XCDs idle at the end of each
    // launch, 87.8 ms against 82.1.
    const int b = deal ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
    int it = 0;
    if (nitems > 1) {
        const int lane = threadIdx.x & 63;
        int count = 0;
        for (int base = 0; base < nitems; base += 64) {
            const int i = base + lane;
            const bool le = i < nitems && gld(&items[i].block_start) <= b;
            count += __popcll(__ballot(le));
        }
        it = __builtin_amdgcn_readfirstlane(count - 1);
    }
    const SliceDesc s = items[it].s;
    TileArgs t = items[it].t;
    t.n = n;
    t.nsteps = TB;
    set_levels(t, s.frame, lv);
    t.ring_lo = ring_lo;
    const int tile = b - items[it].block_start;
    sweep_body<NW, TB, RECOMP>(s, t, deal ? xcd_block(tile, t.ntx * t.ntz * s.nshot) : tile, lds);
}

template <int NW, bool RECOMP>
hipError_t launch_sweep_nw(const SliceDesc *s, const TileArgs *t, const BatchItem *items, int nitems,
                           unsigned blocks, int n, int nsteps, LevelPair lv, int ring_lo, bool deal, hipStream_t st)
{
#define SG_SWEEP(TBV)                                                                                                \
    case TBV:                                                                                                        \
        if (items)                                                                                                   \
            hipLaunchKernelGGL((k_sweep_batch<NW, TBV, RECOMP>), dim3(blocks), dim3(64 * NW), 0, st, items, nitems, \
                               n, lv, ring_lo, deal);                                                                   \
        else                                                                                                         \
            hipLaunchKernelGGL((k_sweep<NW, TBV, RECOMP>), dim3(blocks), dim3(64 * NW), 0, st, *s, *t);            \
        break
    switch (nsteps) {
        SG_SWEEP(1);
        SG_SWEEP(2);
        SG_SWEEP(3);
        SG_SWEEP(4);
        SG_SWEEP(5);
        SG_SWEEP(6);
    default: return hipErrorInvalidValue;
    }
#undef SG_SWEEP
    return hipGetLastError();
}

}  // namespace

Tiling make_sweep_tiling(int Nz, int Nx, int nw, int tb, int seg_h)
{
    Tiling T{};
    T.ex = 64 * nw;
    T.ez = Nz;
    T.k = 0;
    T.tb = tb;
    T.tx = T.ex - 2 * kHalo * tb;
    // equal segments of at most seg_h rows (a short last one leaves its
    // workgroups idle while the others run)
    const int nseg = seg_h > 0 && seg_h < Nz ? (Nz + seg_h - 1) / seg_h : 1;
    T.tz = (Nz + nseg - 1) / nseg;
    T.tz_top = T.tz;          // segments are equal from the top (free top or not)
    T.sweep_nw = nw;
    T.ok = (nw == 2 || nw == 4) && tb >= 1 && tb <= kSweepMaxTimeBlock && T.tx >= 1 && seg_h >= 0;
    if (!T.ok) return T;
    T.ntx = (Nx + T.tx - 1) / T.tx;
    T.ntz = (Nz + T.tz - 1) / T.tz;
    return T;
}

hipError_t launch_sweep(const SliceDesc &s, const TileArgs &t, int nw, hipStream_t st)
{
    const unsigned blocks = (unsigned)(t.ntx * t.ntz * s.nshot);
    const bool ring = t.ring != nullptr;
    switch (nw * 2 + (ring ? 1 : 0)) {
    case 4: return launch_sweep_nw<2, false>(&s, &t, nullptr, 0, blocks, t.n, t.nsteps, {}, 0, false, st);
    case 5: return launch_sweep_nw<2, true>(&s, &t, nullptr, 0, blocks, t.n, t.nsteps, {}, 0, false, st);
    case 8: return launch_sweep_nw<4, false>(&s, &t, nullptr, 0, blocks, t.n, t.nsteps, {}, 0, false, st);
    case 9: return launch_sweep_nw<4, true>(&s, &t, nullptr, 0, blocks, t.n, t.nsteps, {}, 0, false, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sweep_batch(const BatchItem *items, int nitems, int total_blocks, int n, int nsteps,
                              LevelPair lv, int nw, bool deal, hipStream_t st, bool ring, int ring_lo)
{
    const unsigned b = (unsigned)total_blocks;
    switch (nw * 2 + (ring ? 1 : 0)) {
    case 4: return launch_sweep_nw<2, false>(nullptr, nullptr, items, nitems, b, n, nsteps, lv, 0, deal, st);
    case 5: return launch_sweep_nw<2, true>(nullptr, nullptr, items, nitems, b, n, nsteps, lv, ring_lo, deal, st);
    case 8: return launch_sweep_nw<4, false>(nullptr, nullptr, items, nitems, b, n, nsteps, lv, 0, deal, st);
    case 9: return launch_sweep_nw<4, true>(nullptr, nullptr, items, nitems, b, n, nsteps, lv, ring_lo, deal, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace sg
