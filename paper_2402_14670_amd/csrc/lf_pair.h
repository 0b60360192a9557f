// lf_pair.h -- the track kernel body for two input tracks per wavefront.
// Included by lf_kernels.hip (namespace lfk, anonymous).
//
// Lanes 0..31 carry one track, lanes 32..63 the next one, through the steps
// described in lf_kernels.hip, for VELO-UT input seeded in binary32.  The
// arithmetic of every result is the one of Track, in the same order.
//
// The path is bound by vector instruction issue: a plain add, multiply or move
// of registers issues every 2.2 cycles per SIMD, every other vector
// instruction every 4, and the one-track body kept that pipe busy throughout.
// Much of a track's work is the same in every lane (kinematics, list handling)
// or has fewer items than a wavefront has lanes (about 24 seed pairs, 7 kept
// triplets, 2.6 fits), so with 32 lanes per track each of those instructions
// serves two tracks.  What else differs from the one-track body:
//  - windows are padded with +inf, so a sorted search needs no length;
//  - the pairs of all brackets are laid end to end in a queue (92% of them
//    pass the filters), and filter, middle hit and cut run once per pair;
//  - a fit takes four lanes, one per station, instead of sixteen, one per
//    layer: the 2.6 fits of a track fill one pass, and its serial sums need two
//    steps between lanes instead of a transpose through LDS or eleven steps;
//  - in events whose hits lie on the layer planes (EV_PLANES) every expression
//    of the layer z alone is a constant of the context (KParams::lay_*, set_*,
//    fit_tab), and no z or slope is loaded at all;
//  - in the others (PL = false) stereo hits are staged moved along their fibre
//    to the track's y, which is the same for every candidate, and the closest
//    one is found by a search and a short walk.
// Launches before (one track per wavefront) and now: 200,000 nominal tracks
// 0.377 -> 0.226 ms (with sixteen lanes per fit 0.244); 160,000 with per-hit z
// and slopes 0.445 -> 0.250 (0.265); 121,500 in dense events 0.477 -> 0.364
// (0.391); 4,800 nominal 0.0204 -> 0.0160 (0.0199).

// One track's LDS: the x of its window hits (row l: layer l, NW slots, +inf
// past the window's end, so that a sorted search needs no length), per layer
// (u, g(u), dxdy y) and the lists of seeding and candidates.
template <int NW, int MT>
struct alignas(16) HalfLds {
    static constexpr int RS = NW + 1;
    static constexpr int QP = 64;    // queued seed pairs
    uint64_t tk[MT];                 // top-n keys, sorted; ~0 past the list
    int2 win[NL];                    // first hit (event-local) and length of each window
    uint8_t th1[MT];                 // middle hit of each kept triplet
    uint8_t fl[MT];                  // ranks of the candidates to fit
    float4 fit[2];                   // the best candidate: a, b, c, y0; ty, Q, hits
    float4 lay[NL];                  // u, g(u), dxdy * y_ext (0 on x layers), unused
    union {
        struct {
            uint64_t nk[HALF];       // this pass's accepted keys, ~0 past them
            uint16_t q[QP];          // seed pairs: set << 12 | i0 << 6 | i2
        };
        struct {
            float ca[MT], cb[MT], cc[MT];    // triplet x(z) models
            union {
                int8_t ch[MT][NL];           // candidate hits, window-relative, -1 = none
                uint32_t chw[MT][NL / 4];
            };
        };
    };
    float wx[NL * RS];
    float2 zr[2];                    // z range of each seed set's third bucket (hits off the planes)
};

template <int NW, int MT>
struct PairLds {
    HalfLds<NW, MT> h[2];
};

// Entries of a row (non-decreasing, +inf past its end) that satisfy v < x.
template <int NW, class Pred>
__device__ __forceinline__ int row_count(const float *row, Pred pred) {
    int p = 0;
#pragma unroll
    for (int s = NW / 2; s > 0; s >>= 1) p = pred(row[p + s - 1]) ? p + s : p;
    return pred(row[p]) ? p + 1 : p;
}

// Closest entry to xe of row[j] + c given p = #{j: row[j] + c < xe}: the first
// minimum of a linear scan, or -1 (see closest_finish).  p may equal the
// window's length: the +inf there is never closest.
__device__ __forceinline__ int row_closest(const float *row, float c, float xe, int p, float &bd) {
    const int pm = p > 0 ? p - 1 : 0;
    const float d = fabsf(row[p] + c - xe), dl = fabsf(row[pm] + c - xe);
    int best = p;
    bd = d;
    if (!(d < dl)) {
        best = pm;
        bd = dl;
        while (best > 0 && fabsf(row[best - 1] + c - xe) == dl) --best;
    }
    return bd < INFINITY ? best : -1;
}

// The same for a row whose values are out of order by less than W (row[i] <
// row[k] + W for i < k < n): from p, where a search ended, outwards until no
// further value can be as close.  The first minimum of a linear scan.
__device__ __forceinline__ int row_closest_near(const float *row, int n, float xe, float W, int p, float &bd) {
    int best = -1;
    bd = INFINITY;
    for (int i = p - 1; i >= 0; --i) {
        const float v = row[i], d = fabsf(v - xe);
        if (d <= bd) { bd = d; best = i; }
        if (v + W < xe - bd) break;
    }
    for (int i = p; i < n; ++i) {
        const float v = row[i], d = fabsf(v - xe);
        if (d < bd) { bd = d; best = i; }
        if (v - W > xe + bd) break;
    }
    return bd < INFINITY ? best : -1;
}

// (PL: the events' hits lie on the layer planes.)
template <int NW, int MT, bool PL>
struct Pair {
    const DevBatch &B;
    const KParams *__restrict__ P;
    PairLds<NW, MT> &S;
    uint32_t ebase = 0;   // the event's first hit

    static constexpr int RS = HalfLds<NW, MT>::RS;
    static constexpr int QP = HalfLds<NW, MT>::QP;

    // Lane k of each half's value, in every lane of the half.
    __device__ __forceinline__ static int halfmax(int v) {   // v uniform in each half
        const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, HALF);
        return a > b ? a : b;
    }

    // Track tin of the batch (input state) in event ev, result slot t; all
    // uniform in each half; act: the half has a track.
    __device__ __forceinline__ void run(int lane, uint32_t t, uint32_t ev, uint32_t evf, uint32_t tin, bool act) {
        const int j = lane & (HALF - 1);
        HalfLds<NW, MT> &L = S.h[lane >> 5];

        // ---- state, kinematics ----
        const float x_in = B.tx_[tin], y_in = B.ty_[tin], tx_in = B.ttx[tin], ty_in = B.tty[tin];
        const float qop = B.tqop[tin];
        const int l = j < NL ? j : (j < 2 * NL ? j - NL : 0);   // lanes 0..11 and 12..23: layer
        const float zl = P->z[l], dxl = P->dxdy[l];
        const float2 ug = make_float2(P->lay_u[l], P->lay_g[l]);
        const int zone = ty_in >= 0.0f ? 1 : 0;
        ebase = ld32(B.hit_off, ev * 24u);
        const uint32_t b0 = ld32(B.hit_off, ev * 24u + (uint32_t)(2 * l + zone));
        const uint32_t b1 = ld32(B.hit_off, ev * 24u + (uint32_t)(2 * l + zone + 1));
        // the bucket's index, fetched while the bounds are computed
        const BucketIndex *bi = B.bidx + (size_t)(ev * 24u + (uint32_t)(2 * l + zone));
        const bool indexed = B.bidx != nullptr && !(evf & EV_NO_INDEX);
        float ilo = 0.0f, iscale = 0.0f;
        if (indexed) { ilo = bi->lo; iscale = bi->scale; }
        float zlo = 0.0f, zhi = 0.0f, dspread = 0.0f, big = 0.0f;   // the bucket's ranges
        if constexpr (!PL) {
            zlo = bi->zmin;
            zhi = bi->zmax;
            dspread = bi->dspread;
            big = bi->xabs + bi->dabs * fabsf(y_in + ty_in * (zl - P->z_in));
        }
        const float dR = P->dRatio;
        const float p = 1.0f / fabsf(qop);
        const int q = qop > 0.0f ? 1 : -1;
        const float x_mag = x_in + tx_in * (P->z_mag - P->z_in);
        const bool paper = P->field_form == 1;
        float fc[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        float dtx;
        bool live = act;
        if (paper) {
            const float cl = field_c_lane(P, tx_in, ty_in, j);
#pragma unroll
            for (int i = 0; i < 5; ++i) fc[i] = __shfl(cl, (lane & HALF) + i);
            const float si = kick_s(tx_in, ty_in);
            float d = 0.0f;
#pragma unroll
            for (int it = 0; it < 3; ++it) {
                const float sf = si + qop * field_F(fc, d);
                if (!(sf * sf < 1.0f)) live = false;
                d = sf * sqrtf((1.0f + ty_in * ty_in) / (1.0f - sf * sf)) - tx_in;
            }
            dtx = d;
        } else {
            dtx = P->kick * qop;
        }
        const float T = tx_in + dtx;
        const float kd = P->kappa * dtx;
        const float xtol = P->xtol_const + P->xtol_pscale / p;

        // ---- search windows: lane l < 12 searches x_min and the centre of
        // layer l side by side, lane 12 + l its x_max ----
        const bool uvl = is_uv(l);
        const float ye = y_in + ty_in * (zl - P->z_in);
        const float cuv = uvl ? dxl * ye : 0.0f;
        int first, len;
        {
            const float dz = zl - P->z_mag;
            const float dzT = zl - P->z_T;
            const float xe = x_mag + T * dz + kd * dzT * dzT * (1.0f + dR * dzT);
            float xc, xmin, xmax;
            if (uvl) {
                xc = xe - cuv;
                xmin = xc - P->uv_halfwidth;
                xmax = xc + P->uv_halfwidth;
            } else {
                float asymL = 0.0f, asymR = 0.0f;
                if (q * P->polarity > 0) asymR = P->xasym; else asymL = P->xasym;
                xc = xe;
                xmin = xc - xtol - asymL;
                xmax = xc + xtol + asymR;
            }
            const float ka = j < NL ? xmin : next_up(xmax);
            uint32_t la = b0, lc = b0, na = b1 - b0, nc = na;
            if (indexed) {
                const uint16_t *sa = &bi->start[index_cell(ka, ilo, iscale)];
                const uint16_t *sc = &bi->start[index_cell(xc, ilo, iscale)];
                const uint32_t a0 = sa[0], a1 = sa[1], c0 = sc[0], c1 = sc[1];
                la = b0 + a0;
                na = a1 - a0;
                lc = b0 + c0;
                nc = c1 - c0;
            }
            if (!live || j >= 2 * NL) na = 0;
            if (!live || j >= NL) nc = 0;
            while (__ballot((na | nc) != 0)) {
                const uint32_t ha = na >> 1, hc = nc >> 1;
                float va = INFINITY, vc = INFINITY;   // a finished search stays
                if (na) va = ld32(B.hx, la + ha);
                if (nc) vc = ld32(B.hx, lc + hc);
                const bool ta = va < ka, tc = vc < xc;
                la += ta ? ha + 1 : 0;
                na = ta ? na - ha - 1 : ha;
                lc += tc ? hc + 1 : 0;
                nc = tc ? nc - hc - 1 : hc;
            }
            const int lo = (int)(la - ebase);
            int c = (int)(lc - ebase);
            int hi = __shfl(lo, (lane & HALF) + l + NL);
            if (!live) hi = lo;
            hi = hi < lo ? lo : hi;
            c = c < lo ? lo : (c > hi ? hi : c);
            const int N = P->n_hits_window;
            first = lo;
            len = hi - lo;
            if (len > N) {
                first = c - N / 2;
                if (first < lo) first = lo;
                if (first > hi - N) first = hi - N;
                len = N;
            }
            if (j < NL) {
                L.win[j] = make_int2(first, len);
                if constexpr (PL) {
                    L.lay[j] = make_float4(ug.x, ug.y, cuv, 0.0f);
                } else {
                    // how far the moved hits of a stereo bucket can be out of
                    // order: the spread of its slopes times y, and far more
                    // than the rounding of the moved values
                    L.lay[j] = make_float4(ug.x, ug.y, ye, dspread * fabsf(ye) * 1.0001f + (1e-3f + 1e-5f * big));
                    if (j == 8) L.zr[0] = make_float2(zlo, zhi);
                    if (j == 11) L.zr[1] = make_float2(zlo, zhi);
                }
            }
        }
        if (j < MT) L.tk[j] = ~0ull;
        const float T_uv0 = P->T_uv_scale * (fabsf(tx_in) + fabsf(ty_in));
        const float T_uv = T_uv0 < P->T_uv_floor ? P->T_uv_floor : T_uv0;
        wave_sync();

        // ---- stage window hits: round (l, k) brings hits 32 k .. of layer l ----
        {
            constexpr int KR = NW / HALF;
            constexpr int GR = NW == 32 ? 12 : 6;   // layers whose loads are in flight together
#pragma unroll
            for (int l0 = 0; l0 < NL; l0 += GR) {
                float v[GR * KR];
#pragma unroll
                for (int i = 0; i < GR * KR; ++i) {
                    const int2 w = L.win[l0 + i / KR];
                    const int s = j + HALF * (i % KR);
                    v[i] = INFINITY;
                    if (s < w.y) {
                        const uint32_t gi = ebase + (uint32_t)(w.x + s);
                        v[i] = ld32(B.hx, gi);
                        // off the planes a stereo hit is staged moved along its
                        // fibre to the track's y at the layer
                        if constexpr (!PL) {
                            if (is_uv(l0 + i / KR)) v[i] = v[i] + ld32(B.hd, gi) * L.lay[l0 + i / KR].z;
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < GR * KR; ++i)
                    L.wx[(l0 + i / KR) * RS + j + HALF * (i % KR)] = v[i];
            }
            if (j < NL) L.wx[j * RS + NW] = INFINITY;
        }
        wave_sync();

        // ---- seed pairs ----
        // Items: the first-layer hits of both seed sets (set 0, then 1), two
        // per lane; each gets the range of third-layer hits that can pass the
        // magnet filter (the bracket explained in Track::run; here the lever
        // arm and the distance of the planes are the geometry's), and the
        // pairs of all ranges are laid end to end in the queue.
        const float tolc = P->magtol_const + P->magtol_pscale / p;
        const bool low_p = p < P->p_charge_cut;
        int nL = 0;    // kept triplets of this half
        const int c1 = L.win[0].y, n_items = c1 + L.win[3].y;
        const int items_max = halfmax(n_items);
        for (int base = 0; base < items_max; base += 2 * HALF) {
            int jlo[2], cnt[2], code[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int item = base + j + HALF * k;
                const bool s = item >= c1;
                const int i0 = (s ? item - c1 : item) & (NW - 1);
                const float x0 = L.wx[(s ? 3 * RS : 0) + i0];
                const float *row2 = &L.wx[s ? 11 * RS : 8 * RS];
                const int n2 = s ? L.win[11].y : L.win[8].y;
                float xlo, xhi;
                bool all;   // no bracket, or one that overflowed: every pair
                if constexpr (PL) {
                    const float rl = s ? P->set_rlev[1] : P->set_rlev[0];
                    const float dz = s ? P->set_dz[1] : P->set_dz[0];
                    float w0;
                    const float tc = slope_bracket(x0, x_mag, rl, tolc, w0);
                    const float e = x0 + tc * dz;
                    w0 = w0 * dz;
                    const float w = w0 + (0.5f + 2e-5f * (fabsf(e) + w0));
                    xlo = e - w;
                    xhi = e + w;
                    all = !(fabsf(e) + w < 1e30f);
                } else {
                    const float z0 = item < n_items ? ld32(B.hz, ebase + (uint32_t)(L.win[s ? 3 : 0].x + i0)) : 0.0f;
                    const float2 zr = L.zr[s ? 1 : 0];
                    const float lev = P->z_mag - z0, dzl = zr.x - z0, dzh = zr.y - z0;
                    float dt;
                    const float tc = slope_bracket(x0, x_mag, __builtin_amdgcn_rcpf(lev), tolc, dt);
                    // corners of the slope and z intervals
                    const float q1 = (tc - dt) * dzl, q2 = (tc - dt) * dzh;
                    const float q3 = (tc + dt) * dzl, q4 = (tc + dt) * dzh;
                    const float e1 = x0 + fminf(fminf(q1, q2), fminf(q3, q4));
                    const float e2 = x0 + fmaxf(fmaxf(q1, q2), fmaxf(q3, q4));
                    const float margin = 0.5f + 1e-5f * (fabsf(e1) + fabsf(e2));
                    xlo = e1 - margin;
                    xhi = e2 + margin;
                    all = !(fabsf(lev) > 1.0f && (dzl > 1.0f || dzh < -1.0f) && fabsf(xlo) < 1e30f && fabsf(xhi) < 1e30f);
                }
                int lo = row_count<NW>(row2, [xlo](float v) { return v < xlo; });
                int hi = row_count<NW>(row2, [xhi](float v) { return v <= xhi; });
                if (all) { lo = 0; hi = n2; }
                jlo[k] = lo;
                cnt[k] = item < n_items && hi > lo ? hi - lo : 0;
                code[k] = ((s ? 1 : 0) << 12) | (i0 << 6) | lo;
            }
            // offsets: an inclusive scan over the half of both counts at once
            int sc = cnt[0] | (cnt[1] << 16);
            const int own = sc;
            sc += __builtin_amdgcn_update_dpp(0, sc, 0x111, 0xF, 0xF, true);
            sc += __builtin_amdgcn_update_dpp(0, sc, 0x112, 0xF, 0xF, true);
            sc += __builtin_amdgcn_update_dpp(0, sc, 0x114, 0xF, 0xF, true);
            sc += __builtin_amdgcn_update_dpp(0, sc, 0x118, 0xF, 0xF, true);
            sc += __builtin_amdgcn_update_dpp(0, sc, 0x142, 0xA, 0xF, false);   // lane 15 of rows 0, 2 to rows 1, 3
            const int tot2 = __shfl(sc, lane | (HALF - 1));
            const int off0 = (sc - own) & 0xffff, off1 = ((sc - own) >> 16) + (tot2 & 0xffff);
            const int total = (tot2 & 0xffff) + (tot2 >> 16);
            const int total_max = halfmax(total);
            for (int q0 = 0; q0 < total_max; q0 += QP) {
                // queue entries q0 .. q0 + QP of the end-to-end pairs
                for (int k = 0; __ballot(k < cnt[0] || k < cnt[1]); ++k) {
                    const int a0 = off0 + k - q0, a1 = off1 + k - q0;
                    if (k < cnt[0] && (unsigned)a0 < (unsigned)QP) L.q[a0] = (uint16_t)(code[0] + k);
                    if (k < cnt[1] && (unsigned)a1 < (unsigned)QP) L.q[a1] = (uint16_t)(code[1] + k);
                }
                wave_sync();
                const int n_here = total - q0 < QP ? total - q0 : QP;
                const int n_max = total_max - q0 < QP ? total_max - q0 : QP;
                for (int f = 0; f < n_max; f += HALF)
                    triplets(lane, f + j < n_here, L.q[(f + j) & (QP - 1)], nL, tolc, low_p, tx_in, qop, x_mag);
                wave_sync();
            }
        }

        int best_r = -1;    // this half's best candidate
        if (halfmax(nL) > 0) {
            candidates(lane, nL, T_uv);
            best_r = fits(lane, nL, T_uv, y_in, ty_in);
        }

        // ---- output ----
        if (!act) return;
        const bool found = best_r >= 0;
        if (j == 0) {
            const float4 f0 = L.fit[0], f1 = L.fit[1];
            const float bfa = f0.x, bfb = f0.y, bfc = f0.z, bfy0 = f0.w, bfty = f1.x;
            const float uT = P->z_T - P->z_ref;
            const float txT = bfb + 2.0f * bfc * uT + 3.0f * bfc * dR * uT * uT;
            const float qo = paper ? (kick_s(txT, bfty) - kick_s(tx_in, ty_in)) / field_F(fc, txT - tx_in)
                                   : (txT - tx_in) / P->kick;
            B.found[t] = found ? 1 : 0;
            B.nhits[t] = found ? (uint8_t)__float_as_int(f1.z) : 0;
            B.a[t] = found ? bfa : 0.0f;
            B.b[t] = found ? bfb : 0.0f;
            B.c[t] = found ? bfc : 0.0f;
            B.y0[t] = found ? bfy0 : 0.0f;
            B.ty[t] = found ? bfty : 0.0f;
            B.qop[t] = found ? qo : 0.0f;
            B.Q[t] = found ? f1.y : 0.0f;
        }
        if (j < NL) {
            const int h = found ? (int)L.ch[best_r][j] : -1;
            B.hit_idx[(size_t)t * NL + j] = h >= 0 ? first + h : -1;
        }
    }

    // The doublet slopes that can pass the magnet filter lie within dt of the
    // returned one: tolb / |lever arm| with tolb >= the tolerance (rl: 1 / lever
    // arm).
    __device__ __forceinline__ float slope_bracket(float x0, float x_mag, float rl, float tolc, float &dt) const {
        const float arl = fabsf(rl);
        const float tc = (x_mag - x0) * rl;
        const float txs = P->magtol_txscale > 0.0f ? P->magtol_txscale : 0.0f;
        float tolb = tolc + txs * (fabsf(tc) + P->magtol_max * arl);
        if (tolb < P->magtol_min) tolb = P->magtol_min;
        if (tolb > P->magtol_max) tolb = P->magtol_max;
        dt = tolb * arl;
        return tc;
    }

    // Up to 32 seed pairs per half (one per lane, in: the lane has one): the
    // doublet filters, the closest middle hit, the triplet cut, and the merge
    // of the accepted triplets into the half's top-n list.
    __device__ __forceinline__ void triplets(int lane, bool in, uint32_t e, int &nL, float tolc, bool low_p,
                                             float tx_in, float qop, float x_mag) {
        const int j = lane & (HALF - 1);
        HalfLds<NW, MT> &L = S.h[lane >> 5];
        const int NT = P->n_triplets;
        const bool s = (e >> 12) & 1u;
        const int i0 = (int)((e >> 6) & 63u), i2 = (int)(e & 63u);
        const float x0 = L.wx[(s ? 3 * RS : 0) + (i0 & (NW - 1))], x2 = L.wx[(s ? 11 * RS : 8 * RS) + (i2 & (NW - 1))];
        const float z1 = s ? P->z[7] : P->z[4];
        float z0 = s ? P->z[3] : P->z[0], dz = s ? P->set_dz[1] : P->set_dz[0];
        if constexpr (!PL) {
            z0 = in ? ld32(B.hz, ebase + (uint32_t)(L.win[s ? 3 : 0].x + i0)) : 0.0f;
            dz = (in ? ld32(B.hz, ebase + (uint32_t)(L.win[s ? 11 : 8].x + i2)) : 1.0f) - z0;
        }
        const float txd = (x2 - x0) / dz;
        bool ok = in && !(low_p && !((txd - tx_in) * qop > 0.0f));
        const float xm = x0 + txd * (P->z_mag - z0);
        float tol = tolc + P->magtol_txscale * fabsf(txd);
        if (tol < P->magtol_min) tol = P->magtol_min;
        if (tol > P->magtol_max) tol = P->magtol_max;
        if (!(fabsf(xm - x_mag) < tol)) ok = false;
        const float x1e = z1 * txd + (x0 - txd * z0) * (s ? P->K_last : P->K_first);
        const float *row1 = &L.wx[s ? 7 * RS : 4 * RS];
        float bd;
        const int best = row_closest(row1, 0.0f, x1e, row_count<NW>(row1, [x1e](float v) { return v < x1e; }), bd);
        const float chi2 = bd * bd;
        ok = ok && best >= 0 && chi2 < P->T_triplet;
        const uint64_t key = ((uint64_t)__float_as_uint(chi2) << 32) | e;
        // a full list only admits keys below its last one
        ok = ok && key < L.tk[NT - 1];
        const uint64_t bal = __ballot(ok);
        if (bal == 0) return;

        // merge: an element's place is its rank among the kept and the new keys
        const uint32_t mine_bal = lane >= HALF ? (uint32_t)(bal >> HALF) : (uint32_t)bal;
        const int nb = __popc(mine_bal);
        const int nb_max = halfmax(nb), nL_max = halfmax(nL);
        // (the lists are read four keys at a time, past their ends ~0)
        const uint64_t old = L.tk[j & (MT - 1)];
        const int oh1 = L.th1[j & (MT - 1)];
        int r_new = 0, r_old = j;
        L.nk[j] = ~0ull;
        wave_sync();
        if (ok) L.nk[__popc(mine_bal & ((1u << j) - 1u))] = key;
        wave_sync();
        for (int i = 0; i < nb_max; i += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) r_new += L.nk[i + k] < key ? 1 : 0;
        }
        if (nL_max > 0) {
            for (int i = 0; i < nL_max; i += 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) r_new += L.tk[i + k] < key ? 1 : 0;
            }
            for (int i = 0; i < nb_max; i += 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) r_old += L.nk[i + k] < old ? 1 : 0;
            }
        }
        wave_sync();
        if (ok && r_new < NT) {
            L.tk[r_new] = key;
            L.th1[r_new] = (uint8_t)best;
        }
        if (j < nL && r_old < NT) {
            L.tk[r_old] = old;
            L.th1[r_old] = (uint8_t)oh1;
        }
        nL = nL + nb < NT ? nL + nb : NT;
        wave_sync();
    }

    // Triplet x(z) models, one lane per kept triplet, and the extension to
    // the missing layers, two (candidate, layer) items per lane.
    __device__ __forceinline__ void candidates(int lane, int nL, float T_uv) {
        const int j = lane & (HALF - 1);
        HalfLds<NW, MT> &L = S.h[lane >> 5];
        if (j < nL) {
            const uint32_t lo = (uint32_t)L.tk[j];
            const int s = (int)((lo >> 12) & 1u), i0 = (int)((lo >> 6) & 63u), i2 = (int)(lo & 63u);
            const int i1 = L.th1[j];
            const float X0 = L.wx[(s ? 3 * RS : 0) + i0], X1 = L.wx[(s ? 7 * RS : 4 * RS) + i1],
                        X2 = L.wx[(s ? 11 * RS : 8 * RS) + i2];
            float u0, g0, du01, du12, G01, dG;
            if constexpr (PL) {
                u0 = s ? P->lay_u[3] : P->lay_u[0];
                g0 = s ? P->lay_g[3] : P->lay_g[0];
                du01 = s ? P->set_du01[1] : P->set_du01[0];
                du12 = s ? P->set_du12[1] : P->set_du12[0];
                G01 = s ? P->set_G01[1] : P->set_G01[0];
                dG = s ? P->set_dG[1] : P->set_dG[0];
            } else {
                const float dR = P->dRatio;
                u0 = ld32(B.hz, ebase + (uint32_t)(L.win[s ? 3 : 0].x + i0)) - P->z_ref;
                const float u1 = ld32(B.hz, ebase + (uint32_t)(L.win[s ? 7 : 4].x + i1)) - P->z_ref;
                const float u2 = ld32(B.hz, ebase + (uint32_t)(L.win[s ? 11 : 8].x + i2)) - P->z_ref;
                g0 = g_of(u0, dR);
                const float g1 = g_of(u1, dR), g2 = g_of(u2, dR);
                du01 = u1 - u0;
                du12 = u2 - u1;
                G01 = (g1 - g0) / du01;
                dG = (g2 - g1) / du12 - G01;
            }
            const float s01 = (X1 - X0) / du01;
            const float s12 = (X2 - X1) / du12;
            const float c = (s12 - s01) / dG;
            const float b = s01 - c * G01;
            const float a = X0 - b * u0 - c * g0;
            L.ca[j] = a;
            L.cb[j] = b;
            L.cc[j] = c;
            // a seed hit is the first (set 0) or last (set 1) layer of its station
            const uint32_t none = s ? 0x00FFFFFFu : 0xFFFFFF00u;
            const int sh = s ? 24 : 0;
            L.chw[j][0] = none | ((uint32_t)i0 << sh);
            L.chw[j][1] = none | ((uint32_t)i1 << sh);
            L.chw[j][2] = none | ((uint32_t)i2 << sh);
        }
        wave_sync();

        const int n_items = nL * NSLOT, n_max = halfmax(n_items);
        struct Item {
            int r, l;
            bool in, uv;
            float c, xe, W;
            const float *row;
            int n;
        };
        auto item = [&](int it) {
            Item e;
            e.in = it < n_items;
            const int k = e.in ? it : 0;
            e.r = k / NSLOT;
            const int slot = k - NSLOT * (k / NSLOT);
            const int s = (int)(((uint32_t)L.tk[e.r] >> 12) & 1u);
            e.uv = slot >= 3;
            e.l = e.uv ? 4 * ((slot - 3) >> 1) + 1 + ((slot - 3) & 1) : 4 * slot + (s ? 0 : 3);
            const float4 y = L.lay[e.l];
            e.xe = L.ca[e.r] + L.cb[e.r] * y.x + L.cc[e.r] * y.y;
            e.c = PL ? y.z : 0.0f;
            e.row = &L.wx[e.l * RS];
            e.W = 0.0f;
            e.n = 0;
            if constexpr (!PL) {
                e.W = e.uv ? y.w + 1e-6f * fabsf(e.xe) : 0.0f;
                e.n = L.win[e.l].y;
            }
            return e;
        };
        auto closest = [](const Item &e, int p, float &bd) {
            if constexpr (PL) return row_closest(e.row, e.c, e.xe, p, bd);
            else return e.uv ? row_closest_near(e.row, e.n, e.xe, e.W, p, bd) : row_closest(e.row, e.c, e.xe, p, bd);
        };
        auto keep = [&](const Item &e, int best, float bd) {
            if (e.in && best >= 0 && bd * bd < (e.uv ? T_uv : P->T_x)) L.ch[e.r][e.l] = (int8_t)best;
        };
        for (int it = j; it - j < n_max; it += 2 * HALF) {
            const Item a = item(it);
            if (it - j + HALF < n_max) {
                const Item b = item(it + HALF);
                int pa = 0, pb = 0;
#pragma unroll
                for (int s = NW / 2; s > 0; s >>= 1) {
                    const float va = a.row[pa + s - 1] + a.c, vb = b.row[pb + s - 1] + b.c;
                    pa = va < a.xe ? pa + s : pa;
                    pb = vb < b.xe ? pb + s : pb;
                }
                pa = a.row[pa] + a.c < a.xe ? pa + 1 : pa;
                pb = b.row[pb] + b.c < b.xe ? pb + 1 : pb;
                float da, db;
                const int ba = closest(a, pa, da), bb = closest(b, pb, db);
                keep(a, ba, da);
                keep(b, bb, db);
            } else {
                const float c = a.c, xe = a.xe;
                float da;
                const int pa = row_count<NW>(a.row, [c, xe](float v) { return v + c < xe; });
                const int ba = closest(a, pa, da);
                keep(a, ba, da);
            }
        }
        wave_sync();
    }

    // The serial sum over the 12 layers of a candidate, ((+0 + t_0) + t_1) + ...,
    // from the n terms each of a quad's lanes 0..2 holds of its station (in
    // layer order): every lane adds its terms three times, starting from +0 and
    // then from the lane before it, so that lane 2 ends with the whole sum,
    // which the quad receives.
    template <int N>
    __device__ __forceinline__ static float quad_sum(const float (&t)[N]) {
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < N; ++i) s = s + t[i];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            s = quad<0x90>(s);   // from the lane before (lane 0: its own)
#pragma unroll
            for (int i = 0; i < N; ++i) s = s + t[i];
        }
        return quad<0xAA>(s);
    }
    template <int PERM>
    __device__ __forceinline__ static float quad(float v) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), PERM, 0xF, 0xF, true));
    }
    template <int PERM>
    __device__ __forceinline__ static uint32_t quad(uint32_t v) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, PERM, 0xF, 0xF, true);
    }

    // Fits and quality: four lanes per candidate, eight candidates of each
    // track per pass in rank order.  Lanes 0..2 of a quad hold the four layers
    // (x u v x) of a station each, so a sum over the layers is two steps
    // between lanes, and the x and stereo formulas need no selection.  The
    // sums of the layer terms alone depend only on which layers have a hit:
    // FitRow of that 12-bit mask, tabulated per context (hits on the planes).
    // Returns the half's best candidate (its fit is in fit[]), or -1.
    __device__ __forceinline__ int fits(int lane, int nL, float T_uv, float y_in, float ty_in) {
        const int j = lane & (HALF - 1);
        HalfLds<NW, MT> &L = S.h[lane >> 5];
        uint32_t mine;   // the half's candidates to fit
        {
            bool rule = false;
            if (j < nL) {
                int n = 0;
                bool st_ok = true;
#pragma unroll
                for (int st = 0; st < 3; ++st) {
                    const uint32_t pres = ~L.chw[j][st] & 0x80808080u;
                    n += __popc(pres);
                    st_ok = st_ok && (pres & 0x00808000u) != 0u;
                }
                rule = n >= 9 && st_ok;
            }
            const uint64_t bal = __ballot(rule);
            mine = lane >= HALF ? (uint32_t)(bal >> HALF) : (uint32_t)bal;
            if (rule) L.fl[__popc(mine & ((1u << j) - 1u))] = (uint8_t)j;
        }
        const int nf = __popc(mine), nf_max = halfmax(nf);
        wave_sync();
        int best_r = -1;
        float best_Q = 0.0f;
        const int st = j & 3, sq = st < 3 ? st : 0;   // lane 3 holds no layers
        const float dR = P->dRatio;
        float u[4], gu[4], sv[4], h[4], cuv[2], dxy[2];
        if constexpr (PL) {
            const float4 u4 = *reinterpret_cast<const float4 *>(&P->lay_u[4 * sq]);
            const float4 g4 = *reinterpret_cast<const float4 *>(&P->lay_g[4 * sq]);
            const float4 s4 = *reinterpret_cast<const float4 *>(&P->lay_s[4 * sq]);
            const float4 h4 = *reinterpret_cast<const float4 *>(&P->lay_h[4 * sq]);
            u[0] = u4.x; u[1] = u4.y; u[2] = u4.z; u[3] = u4.w;
            gu[0] = g4.x; gu[1] = g4.y; gu[2] = g4.z; gu[3] = g4.w;
            sv[0] = s4.x; sv[1] = s4.y; sv[2] = s4.z; sv[3] = s4.w;
            h[0] = h4.x; h[1] = h4.y; h[2] = h4.z; h[3] = h4.w;
            cuv[0] = L.lay[4 * sq + 1].z; cuv[1] = L.lay[4 * sq + 2].z;
            dxy[0] = P->dxdy[4 * sq + 1]; dxy[1] = P->dxdy[4 * sq + 2];
        }
        for (int f0 = 0; f0 < nf_max; f0 += HALF / 4) {
            const int k = f0 + (j >> 2);
            const bool on = k < nf;
            const int r = on ? (int)L.fl[k] : 0;
            const float a = L.ca[r], b = L.cb[r], c = L.cc[r];
            const uint32_t word = on && st < 3 ? L.chw[r][sq] : ~0u;
            const uint32_t absent = word & 0x80808080u;
            // the layers with a hit: four bits per station
            uint32_t mask = (((~word & 0x80808080u) * 0x204081u) >> 28) << (4 * sq);
            mask |= quad<0xB1>(mask);   // lanes 1 0 3 2
            mask |= quad<0x4E>(mask);   // lanes 2 3 0 1
            const FitRow *Ft = P->fit_tab + mask;
            FitRow F;
            if constexpr (PL) F = *Ft;
            float rr[4], R0, R1, R2;
            bool pres[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pres[i] = !(absent & (0x80u << (8 * i)));
                const int hit = (int)((word >> (8 * i)) & 0x7Fu);
                const bool st_layer = i == 1 || i == 2;
                float xm = 0.0f;
                if constexpr (PL) {
                    // (an absent hit reads within the row and is dropped)
                    xm = L.wx[(4 * sq + i) * RS + (hit & (NW - 1))];
                    if (st_layer) xm = xm + cuv[i - 1];
                } else {
                    u[i] = sv[i] = h[i] = gu[i] = 0.0f;
                    if (st_layer) dxy[i - 1] = 1.0f;
                    if (pres[i]) {
                        const uint32_t gi = ebase + (uint32_t)(L.win[4 * sq + i].x + hit);
                        const float x = ld32(B.hx, gi), z = ld32(B.hz, gi);
                        u[i] = z - P->z_ref;
                        xm = x;
                        if (st_layer) {
                            dxy[i - 1] = ld32(B.hd, gi);
                            xm = x + dxy[i - 1] * (y_in + ty_in * (z - P->z_in));
                        }
                        sv[i] = u[i] * INV1024;
                        h[i] = sv[i] * sv[i] * (1.0f + dR * u[i]);
                        gu[i] = g_of(u[i], dR);
                    }
                }
                const float m = xm - (a + b * u[i] + c * gu[i]);
                rr[i] = pres[i] ? m : 0.0f;
            }
            if constexpr (!PL) {
                const float q0[4] = {sv[0], sv[1], sv[2], sv[3]}, q1[4] = {h[0], h[1], h[2], h[3]};
                const float q2[4] = {sv[0] * sv[0], sv[1] * sv[1], sv[2] * sv[2], sv[3] * sv[3]};
                const float q3[4] = {sv[0] * h[0], sv[1] * h[1], sv[2] * h[2], sv[3] * h[3]};
                const float q4[4] = {h[0] * h[0], h[1] * h[1], h[2] * h[2], h[3] * h[3]};
                const float q5[2] = {sv[1], sv[2]}, q6[2] = {q2[1], q2[2]};
                F.S1 = quad_sum(q0);
                F.S2 = quad_sum(q1);
                F.S11 = quad_sum(q2);
                F.S12 = quad_sum(q3);
                F.S22 = quad_sum(q4);
                F.YS1 = quad_sum(q5);
                F.YS11 = quad_sum(q6);
                F.S0 = (float)__popc(mask);
                F.YS0 = (float)__popc(mask & 0x666u);   // the stereo layers 1, 2, 5, 6, 9, 10
                F.m00 = F.S11 * F.S22 - F.S12 * F.S12;
                F.m01 = F.S1 * F.S22 - F.S12 * F.S2;
                F.m02 = F.S1 * F.S12 - F.S11 * F.S2;
                F.det = F.S0 * F.m00 - F.S1 * F.m01 + F.S2 * F.m02;
                F.D = F.YS0 * F.YS11 - F.YS1 * F.YS1;
                F.C = Ft->C;
            }
            {
                const float q1[4] = {sv[0] * rr[0], sv[1] * rr[1], sv[2] * rr[2], sv[3] * rr[3]};
                const float q2[4] = {h[0] * rr[0], h[1] * rr[1], h[2] * rr[2], h[3] * rr[3]};
                R0 = quad_sum(rr);
                R1 = quad_sum(q1);
                R2 = quad_sum(q2);
            }
            const bool ok_x = fabsf(F.det) > 0.0f;
            const float det_s = ok_x ? F.det : 1.0f;
            // lanes 0, 1 and 2 divide the numerators of da, db and dc
            const float A = R1 * F.S22 - F.S12 * R2, E = R1 * F.S12 - F.S11 * R2, G = F.S1 * R2 - R1 * F.S2;
            const float num_x = st == 0 ? R0 * F.m00 - F.S1 * A + F.S2 * E
                              : st == 1 ? F.S0 * A - R0 * F.m01 + F.S2 * G
                                        : F.S0 * (F.S11 * R2 - R1 * F.S12) - F.S1 * G + R0 * F.m02;
            const float q_x = num_x / det_s;
            const float da = quad<0x00>(q_x), db = quad<0x55>(q_x), dc = quad<0xAA>(q_x);
            float chi[4], eta[2], eta_s[2];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool st_layer = i == 1 || i == 2;
                const float res = rr[i] - (da + db * sv[i] + dc * h[i]);
                const float q = res * res / (st_layer ? T_uv : P->T_x);
                chi[i] = pres[i] ? q : 0.0f;
                if (st_layer) {
                    const float y = -res / dxy[i - 1];
                    eta[i - 1] = pres[i] ? y : 0.0f;
                    eta_s[i - 1] = sv[i] * eta[i - 1];
                }
            }
            const float Qx = quad_sum(chi), Y0 = quad_sum(eta), Y1 = quad_sum(eta_s);
            const bool ok_y = fabsf(F.D) > 0.0f;
            const float D_s = ok_y ? F.D : 1.0f;
            const float q_y = (st == 0 ? Y0 * F.YS11 - F.YS1 * Y1 : F.YS0 * Y1 - F.YS1 * Y0) / D_s;   // dy0, dty
            const float dy0 = quad<0x00>(q_y), dty = quad<0x55>(q_y);
            const float dslope = dty * INV1024;
            float chy[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float ry = eta[i] - (dy0 + dty * sv[i + 1]);
                const float q = ry * ry / P->T_y;
                chy[i] = pres[i + 1] ? q : 0.0f;
            }
            const float Qy = quad_sum(chy);
            const float q_q = (st == 0 ? Qx : Qy) / (st == 0 ? F.S0 - 3.0f : F.YS0 - 2.0f);
            const float Q = (quad<0x00>(q_q) + quad<0x55>(q_q)) * F.C;
            const bool acc = on && ok_x && ok_y && fabsf(dslope) < P->T_ty && Q < P->T_Q;
            // the half's least Q; of equal ones the lowest rank (lane)
            float m = acc ? Q : INFINITY;
            m = fminf(m, dpp<0x124, false>(m));   // row_ror:4
            m = fminf(m, dpp<0x128, false>(m));   // row_ror:8
            m = fminf(m, __shfl_xor(m, 16));
            const uint64_t bal = __ballot(acc && Q == m);
            const uint32_t at = lane >= HALF ? (uint32_t)(bal >> HALF) : (uint32_t)bal;
            if (at != 0u && (best_r < 0 || m < best_Q)) {
                const int wl = __builtin_ctz(at);
                best_r = (int)L.fl[f0 + (wl >> 2)];
                best_Q = m;
                if (j == wl) {
                    L.fit[0] = make_float4(a + da, b + db * INV1024, c + dc * INV1024SQ,
                                           (y_in + ty_in * (P->z_ref - P->z_in)) + dy0);
                    L.fit[1] = make_float4(ty_in + dslope, Q, __int_as_float(__popc(mask)), 0.0f);
                }
            }
        }
        wave_sync();
        return best_r;
    }
};
