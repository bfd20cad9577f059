// fdw_stream_rows.h - one block of U rows of a streaming work item: the body of the row loop of
// sweep_item (fdw_stream.h), whose names it uses.  It stands in two places there and is a file of its own
// because the two cost different registers.  Most variants have it in a function object, which can
// shorten the first block (HEAD), and are as fast or faster that way (FP32 time block 7 with energies at
// 1200^2, 84 steps: 332 us, 370 in the loop).  In FP32 with faces and energies the object takes 173
// registers instead of 166, beyond the 168 of three waves per SIMD (1531 x 1177, 80 steps: 426 us as an
// object, 351 in the loop), and 262 instead of 253 with 4 columns per lane at time block 6, beyond the 256
// of two (1500^2, 96 steps: 678 and 515): these have it in the loop itself.
{
    T eb[K];
#pragma unroll
    for (int t = 0; t < K; ++t) eb[t] = T(0);
#pragma unroll
    for (int s = 0; s < U; ++s) {
        const int p = blk * U + s;  // stream position of the row loaded last
        const int pb = s % NB;      // buffer holding row p
        // prefetch row p+NB-1 into the buffer row p-1 used
        {
            const int pn = (s + NB - 1) % NB;
            load_row(p + NB - 1, bu[pn], bd[pn], bh[pn], bhy[pn]);
        }

        // ---- coefficient faces of row p-1 into the ring (index (p-1) mod K), scaled
        // by tau^2/(2 dx^2) and tau^2/(2 dy^2) once per row, so that every level's
        // operator is the plain sum of its x and y flux differences; the y face between
        // rows p-1 and p is stored with the upper of the two grid rows
        {
            const int q = pmod(s - 1, K);
            if (FACE) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    FXr[q][c] = ax * hprev[c];
                    FYr[q][c] = ay * ((dir > 0) ? hyprev[c] : bhy[pb][c]);
                    hprev[c] = bh[pb][c];
                    hyprev[c] = bhy[pb][c];
                }
            } else {
                const T hr = lane_from_right(hprev[0]);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    FXr[q][c] = ax * (hprev[c] + ((c < C - 1) ? hprev[c + 1] : hr));
                    FYr[q][c] = ay * (hprev[c] + bh[pb][c]);
                }
#pragma unroll
                for (int c = 0; c < C; ++c) hprev[c] = bh[pb][c];
            }
        }
        // ---- level 0: row p of the input state
        {
            const int p0 = pmod(s, 2);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                Ur[0][p0][c] = bu[pb][c];
                Dr[0][p0][c] = bd[pb][c];
            }
        }
        // ---- levels 1..K
#pragma unroll
        for (int t = 1; t <= K; ++t) {
            if (HEAD && 2 * t - 1 > s) break;
            const int r = rfirst + dir * (p - t);  // grid row of stream position p - t
            const int pr = pmod(s - t, 2);         // parity index of row r
            const int pr1 = pmod(s - t + 1, 2);    // ... of the next row in the stream, r + dir
            const int q = pmod(s - t, K);          // coefficient ring index of row r
            const bool rin = (r >= 1) && (r <= ny - 2);
            const bool rown = !HEAD && (r >= r0) && (r < r1);
            const T right = lane_from_right(Ur[t - 1][pr][0]);
            T F[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T ue = (c < C - 1) ? Ur[t - 1][pr][c + 1] : right;
                F[c] = FXr[q][c] * (ue - Ur[t - 1][pr][c]);
            }
            const T Fl = lane_from_left(F[C - 1]);
            T nu[C], nd[C], L[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                // Gn = fy (u_{r+dir} - u_r): downwards this is F_{r+1/2}, upwards it is
                // -F_{r-1/2} exactly (negation is exact), and Gy holds the previous
                // row's Gn; so Gn - Gy is F_{r+1/2} - F_{r-1/2} bit for bit in both
                // directions
                const T Gn = FYr[q][c] * (Ur[t - 1][pr1][c] - Ur[t - 1][pr][c]);
                const T sx = F[c] - ((c > 0) ? F[c - 1] : Fl);
                const T sy = Gn - Gy[t - 1][c];
                Gy[t - 1][c] = Gn;
                L[c] = sx + sy;
            }
            // Dirichlet rows keep du = 0 (and with it u = 0, which they hold at every
            // level); the row test is wave-uniform, and the empty asm keeps it a scalar
            // branch instead of a select per value
#pragma unroll
            for (int c = 0; c < C; ++c) nd[c] = fma_t(L[c], colm[c], Dr[t - 1][pr][c]);
            if (__builtin_expect(!rin, 0)) {
#pragma unroll
                for (int c = 0; c < C; ++c) nd[c] = T(0);
                asm volatile("");
            }
#pragma unroll
            for (int c = 0; c < C; ++c) nu[c] = Ur[t - 1][pr][c] + nd[c];
            if (want_energy && rown) {
                // per-node terms du^2 - u L in the storage type, summed over the lane's
                // columns and the rows of this unrolled block; FP64 across blocks
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    eb[t - 1] = fma_t(nd[c], nd[c], eb[t - 1]);
                    eb[t - 1] = fma_t(-nu[c], L[c], eb[t - 1]);
                }
                // an empty asm that reads and writes the partial sum pins the
                // accumulation here: otherwise the compiler defers the energy
                // arithmetic of the whole unrolled block to its end, keeping every
                // level's nu, nd and L of every row alive (several hundred registers
                // at K >= 3)
                asm volatile("" : "+v"(eb[t - 1]));
            }
            if (want_trace && !HEAD && __builtin_expect(item_rec, 0)) {
                // receivers of row r in this strip's owned columns, looked up once when
                // the row enters level 1 (none for rows the item does not own or that lie
                // on the boundary), and entered in the row's slots
                if (t == 1) {
                    int kb = 0, ke = 0;
                    bool search = rown && rin;
                    if (pre_item && search) {
                        // the item's row mask: no receivers, or slots looked up already
                        const int ri = r - r0;
                        const uint64_t m = (ri < kWaveSize) ? rmask0 : rmask1;
                        const int b = ri & (kWaveSize - 1);
                        search = false;
                        if ((m >> b) & 1) {
                            const int j = ((ri < kWaveSize) ? 0 : rrank1) + __popcll(m & ((uint64_t(1) << b) - 1));
                            if (j < kPreRows) {
#pragma unroll
                                for (int c = 0; c < C; ++c) s_slot[wib][q][lane * C + c] = s_pre[wib][j][lane * C + c];
                                kb = 0;
                                ke = 1;
                            } else {
                                search = true;
                            }
                        }
                    }
                    if (search) {
                        kb = rowptr[r];
                        ke = rowptr[r + 1];
                        if (kb < ke) {
                            kb = lower_bound_col(rcol, kb, ke, own_lo);
                            ke = lower_bound_col(rcol, kb, ke, own_lo + Wv);
                        }
                        for (int k = kb; k < ke; ++k) {
                            const int col = rcol[k];
                            if ((k == kb || rcol[k - 1] != col) && lane == 0) s_slot[wib][q][col - own_lo + Hx] = rid[k];
                        }
                    }
                    RPb[q] = kb;
                    RPe[q] = ke;
                }
                if (RPb[q] < RPe[q]) {
                    const int64_t row = n0 + t;
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const int id = s_slot[wib][q][lane * C + c];
                        if (id >= 0 && row < trace_rows) trace_out[row * trace_R + id] = nu[c];
                        if (t == K) s_slot[wib][q][lane * C + c] = -1;
                    }
                }
            }
            if (t < K) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    Ur[t][pr][c] = nu[c];
                    Dr[t][pr][c] = nd[c];
                }
            } else if (rown && lane_owned) {
                const size_t off = (size_t)(ptrdiff_t)r * ld + lane_off;
                if (nt) {
                    store_row_nt<T, C>(uout + off, nu);
                    store_row_nt<T, C>(dout + off, nd);
                } else {
                    store_pack<T, C>(uout + off, nu);
                    store_pack<T, C>(dout + off, nd);
                }
            }
        }
        // keep the scheduler from interleaving consecutive rows (bounds register pressure)
        __builtin_amdgcn_sched_barrier(0);
    }
    if (want_energy && !HEAD && lane_owned) {
#pragma unroll
        for (int t = 0; t < K; ++t) acc[t] += (double)eb[t];
    }
}
