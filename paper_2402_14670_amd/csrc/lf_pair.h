// lf_pair.h -- the track kernel body for two input tracks per wavefront.
// Included by lf_kernels.hip (namespace lfk, anonymous).
//
// Lanes 0..31 carry one track, lanes 32..63 the next one, through the steps
// described in lf_kernels.hip, for VELO-UT input (VELO-only input: each half one
// side of the same track).  The arithmetic of every result
// is the one of Track, in the same order.
//
// The path is bound by vector instruction issue: a plain add, multiply or move
// of registers issues every 2.2 cycles per SIMD, every other vector
// instruction every 4, and the one-track body kept that pipe busy throughout.
// Much of a track's work is the same in every lane (kinematics, list handling)
// or has fewer items than a wavefront has lanes (about 24 seed pairs, 7 kept
// triplets, 2.6 fits), so with 32 lanes per track each of those instructions
// serves two tracks.  What else differs from the one-track body:
//  - windows are padded with +inf, so a sorted search needs no length;
//  - the pairs of all brackets are laid end to end over the lanes (92% of them
//    pass the filters), and filter, middle hit and cut run once per pair;
//  - a fit takes four lanes, one per station, instead of sixteen, one per
//    layer: the 2.6 fits of a track fill one pass, and its serial sums need two
//    steps between lanes instead of a transpose through LDS or eleven steps;
//  - likewise a candidate's model and extension: a lane searches its station's
//    three layers side by side, and 16 candidates of both tracks share a pass;
//  - a division whose divisor is a constant of the context multiplies by its
//    binary64 reciprocal (div_by: 15 cycles of issue instead of 38);
//  - in events whose hits lie on the layer planes (not EV_OFF_PLANES) every
//    expression of the layer z alone is a constant of the context
//    (KParams::lay_*, set_*, fit_tab), and no z or slope is loaded at all;
//  - in the others (PL = false) stereo hits are staged moved along their fibre
//    to the track's y, which is the same for every candidate, and the closest
//    one is found by a search and a short walk.
// Launches with one track per wavefront and now: 200,000 nominal tracks 0.383
// -> 0.201 ms (0.244 with the one-track body's sixteen lanes per fit and nine
// lanes per extension, 0.226 with four lanes per fit); 160,000 with per-hit z
// and slopes 0.443 -> 0.228; 121,500 in dense events 0.488 -> 0.276 (0.314 with
// the pairs written into a queue item by item); 100,000 VELO-only 0.471 ->
// 0.305; 160,000 nominal seeded in binary16 0.363 -> 0.180; 4,800 nominal 0.0207 -> 0.0156.

// Binary16 seeding: per track and seed set, coordinates relative to the
// window centres c and the constants rounded once from binary32, as in
// Track::run, and what the bracket of the third layer needs in binary32.
struct alignas(16) SeedSet16 {
    float c[3];        // window centres of the set's layers
    uint32_t on;       // each outer window's hits share one z (else binary32)
    float E0, C02, rs, S;   // E0, C02; 1 / (RZ L0) and |RZ L0|
    float rL, err;     // 1 / |L0|, and the part of the rounding bound common to all pairs
    _Float16 hE0, hC02, hRZ, hL0, hA, hKK, hB, pad;
    uint32_t pad2[2];
};

// One track's LDS: the x of its window hits (row l: layer l, NW slots, +inf
// past the window's end, so that a sorted search needs no length), per layer
// (u, g(u), dxdy y) and the lists of seeding and candidates.
template <int NW, int MT>
struct alignas(16) HalfLds {
    static constexpr int RS = NW + 1;
    uint64_t tk[MT];                 // top-n keys, sorted; ~0 past the list
    int2 win[NL];                    // first hit (event-local) and length of each window
    uint8_t th1[MT];                 // middle hit of each kept triplet
    uint8_t fl[MT];                  // ranks of the candidates to fit
    float4 fit[2];                   // the best candidate: a, b, c, y0; ty, Q, hits
    float4 lay[NL];                  // u, g(u), dxdy * y_ext (0 on x layers), h; off the planes y_ext, slack
    union {
        struct {
            union {
                uint32_t mark[HALF]; // where the items' pairs begin in a pass
                uint64_t nk[HALF];   // its accepted keys, ~0 past them
            };
            SeedSet16 h16[2];        // (binary16 seeding)
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
    float4 set[2][3];                // KParams::set_tab
    double2 rset[2][2];              // KParams::r_set
};

// Rows are searched by LDS byte address: a probe at a fixed distance is an
// offset of the load, and a step is one add, one compare and one select.
typedef __attribute__((address_space(3))) const float lds_float;
__device__ __forceinline__ uint32_t lds_addr(const float *p) {
    return (uint32_t)reinterpret_cast<uintptr_t>((lds_float *)p);
}
__device__ __forceinline__ float lds_at(uint32_t a) { return *reinterpret_cast<lds_float *>((uintptr_t)a); }

// Address of the first entry of a row (non-decreasing, +inf past its end) that
// does not satisfy pred, for N rows side by side.
template <int NW, int N, class Pred>
__device__ __forceinline__ void row_lower(uint32_t (&p)[N], Pred pred) {
#pragma unroll
    for (int s = NW / 2; s > 0; s >>= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const bool t = pred(i, lds_at(p[i] + 4u * (uint32_t)(s - 1)));
            p[i] = t ? p[i] + 4u * (uint32_t)s : p[i];
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const bool t = pred(i, lds_at(p[i]));
        p[i] = t ? p[i] + 4u : p[i];
    }
}

// Closest entry to xe of a row's values + c, given the address p of the first
// value + c not below xe (one past the row's last slot at most: there +inf is
// never closest): the address of the first minimum of a linear scan and its
// distance, or a distance of +inf or NaN (see closest_finish).
__device__ __forceinline__ uint32_t row_closest(uint32_t row, float c, float xe, uint32_t p, float &bd) {
    const uint32_t pm = p > row ? p - 4u : row;
    const float d = fabsf(lds_at(p) + c - xe), dl = fabsf(lds_at(pm) + c - xe);
    const bool left = !(d < dl);
    uint32_t best = left ? pm : p;
    bd = left ? dl : d;
    // equal distances before the left neighbour
    if (left)
        while (best > row && fabsf(lds_at(best - 4u) + c - xe) == dl) best -= 4u;
    return best;
}

// The same for a row whose values are out of order by less than W (row[i] <
// row[k] + W for i < k < n): from p, where a search ended, outwards until no
// further value can be as close.  The first minimum of a linear scan.
__device__ __forceinline__ uint32_t row_closest_near(uint32_t row, uint32_t end, float xe, float W, uint32_t p,
                                                     float &bd) {
    uint32_t best = row;
    bd = INFINITY;
    for (uint32_t i = p; i > row;) {
        i -= 4u;
        const float v = lds_at(i), d = fabsf(v - xe);
        if (d <= bd) { bd = d; best = i; }
        if (v + W < xe - bd) break;
    }
    for (uint32_t i = p; i < end; i += 4u) {
        const float v = lds_at(i), d = fabsf(v - xe);
        if (d < bd) { bd = d; best = i; }
        if (v - W > xe + bd) break;
    }
    return best;
}

// PL: the events' hits lie on the layer planes.  NS = 2 (VELO-only input, two
// windows per layer): one track per wavefront, a half for each side's windows,
// seeds and candidates; the halves meet where the top-n pool of both sides is
// cut and where the best candidate is chosen.
template <int NW, int MT, bool PL, int NS, bool H16 = false>
struct Pair {
    static_assert(NS == 1 || !H16, "binary16 seeding has one window per layer");
    using Half = HalfLds<NW, MT>;
    const DevBatch &B;
    const KParams *__restrict__ P;
    PairLds<NW, MT> &S;
    uint32_t ebase = 0;   // the event's first hit

    static constexpr int RS = Half::RS;

    __device__ __forceinline__ static uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
    __device__ __forceinline__ static int halfmax(int v) {   // v uniform in each half
        const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, HALF);
        return a > b ? a : b;
    }

    // Track tin of the batch (input state) in event ev, result slot t; all
    // uniform in each half (NS = 2: in the wave); act: the half has a track.
    __device__ __forceinline__ void run(int lane, uint32_t t, uint32_t ev, uint32_t evf, uint32_t tin, bool act) {
        const int j = lane & (HALF - 1);
        Half &L = S.h[lane >> 5];

        // ---- state, kinematics ----
        const float x_in = B.tx_[tin], y_in = B.ty_[tin], tx_in = B.ttx[tin], ty_in = B.tty[tin];
        const float qop = B.tqop[tin];
        const int l = j < NL ? j : (j < 2 * NL ? j - NL : 0);   // lanes 0..11 and 12..23: layer
        const float zl = P->z[l], dxl = P->dxdy[l];
        const float4 lz = make_float4(P->lay_u[l], P->lay_g[l], 0.0f, P->lay_h[l]);
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
        float p;
        int q = 0;
        if constexpr (NS == 2) {   // the assumed minimum momentum (Track::run)
            const float t2 = tx_in * tx_in + ty_in * ty_in;
            const float sin_t = sqrtf(t2 / (1.0f + t2));
            const float p_pt = sin_t > 0.0f ? P->noUT_pt_min / sin_t : 0.0f;
            p = p_pt > P->noUT_p_min ? p_pt : P->noUT_p_min;
        } else {
            p = 1.0f / fabsf(qop);
            q = qop > 0.0f ? 1 : -1;
        }
        const float x_mag = x_in + tx_in * (P->z_mag - P->z_in);
        const bool paper = P->field_form == 1;
        float fc[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        float dtx = 0.0f;
        bool live = act;
        if (paper) {
            const float cl = field_c_lane(P, tx_in, ty_in, j);
#pragma unroll
            for (int i = 0; i < 5; ++i) fc[i] = __shfl(cl, (lane & HALF) + i);
            if constexpr (NS == 1) {
                const float si = kick_s(tx_in, ty_in);
                float d = 0.0f;
#pragma unroll
                for (int it = 0; it < 3; ++it) {
                    const float sf = si + qop * field_F(fc, d);
                    if (!(sf * sf < 1.0f)) live = false;
                    d = sf * sqrtf((1.0f + ty_in * ty_in) / (1.0f - sf * sf)) - tx_in;
                }
                dtx = d;
            }
        } else {
            dtx = P->kick * qop;
        }
        const float T = tx_in + dtx;
        const float kd = P->kappa * dtx;
        float xtol;
        if constexpr (NS == 2) {
            const float ip = 1.0f / p;
            const float ty2 = ty_in * ty_in;
            const float *c8 = P->noUT_c;
            xtol = ip * (c8[0] + tx_in * (c8[1] + c8[2] * tx_in) + ty2 * (c8[3] + tx_in * (c8[4] + c8[5] * tx_in)) +
                         ip * (c8[6] * tx_in + c8[7] * ip));
        } else {
            xtol = P->xtol_const + P->xtol_pscale / p;
        }

        // ---- search windows: lane l < 12 searches x_min and the centre of
        // layer l side by side, lane 12 + l its x_max ----
        // the set constants, one run of 40 words in both places
        static_assert(offsetof(KParams, r_set) == offsetof(KParams, set_tab) + 96, "set_tab and r_set are one run");
        if (lane < 40) reinterpret_cast<float *>(&S.set[0][0])[lane] = (&P->set_tab[0][0])[lane];
        const bool uvl = is_uv(l);
        const float ye = y_in + ty_in * (zl - P->z_in);
        const float cuv = uvl ? dxl * ye : 0.0f;
        int first, len;
        float xc;   // lane l: the window centre of layer l
        {
            float xmin, xmax;
            if constexpr (NS == 2) {
                // straight line; two windows per layer sharing an overlap
                const float xe = x_in + tx_in * (zl - P->z_in);
                const float x0 = uvl ? xe - cuv : xe;
                const float tol = uvl ? P->uv_halfwidth : xtol;
                xmin = x0 - (lane < HALF ? tol : P->noUT_overlap);
                xmax = x0 + (lane < HALF ? P->noUT_overlap : tol);
                xc = 0.5f * (xmin + xmax);
            } else {
                const float dz = zl - P->z_mag;
                const float dzT = zl - P->z_T;
                const float xe = x_mag + T * dz + kd * dzT * dzT * (1.0f + dR * dzT);
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
            // Both searches in the same steps s = 2^k .. 1, from the largest any
            // lane needs: the start advances by s while the entry before it
            // stays below the key.
            const uint32_t most = na > nc ? na : nc;
            uint32_t s = 1;
            while (__ballot(most >= 2 * s)) s *= 2;
            const uint32_t ea = la + na, ec = lc + nc;
            for (; s > 0; s >>= 1) {
                const float *at = B.hx + (s - 1);
                const uint32_t ta = la + s, tc = lc + s;
                float va = INFINITY, vc = INFINITY;
                if (ta <= ea) va = ld32(at, la);
                if (tc <= ec) vc = ld32(at, lc);
                la = va < ka ? ta : la;
                lc = vc < xc ? tc : lc;
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
                    L.lay[j] = make_float4(lz.x, lz.y, cuv, lz.w);
                } else {
                    // how far the moved hits of a stereo bucket can be out of
                    // order: the spread of its slopes times y, and far more
                    // than the rounding of the moved values
                    L.lay[j] = make_float4(lz.x, lz.y, ye, dspread * fabsf(ye) * 1.0001f + (1e-3f + 1e-5f * big));
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
        // pairs of all ranges are laid end to end: side << 13 | set << 12 |
        // i0 << 6 | i2.
        const float tolc = P->magtol_const + P->magtol_pscale / p;
        const bool low_p = NS == 1 && p < P->p_charge_cut;
        if constexpr (H16) {
            seeds16(lane, xc, x_mag, tolc);
            wave_sync();
        }
        int nA = 0, nB = 0;    // kept triplets of the two halves (uniform)
        const int c1 = L.win[0].y, n_items = c1 + L.win[3].y;
        const int items_max = halfmax(n_items);
        for (int base = 0; base < items_max; base += 2 * HALF) {
            int cnt[2], code[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int item = base + j + HALF * k;
                const bool s = item >= c1;
                const int i0 = (s ? item - c1 : item) & (NW - 1);
                const int ro = s ? 3 * RS : 0;   // the set's rows: layers 0, 4, 8 or three further
                const float x0 = L.wx[ro + i0];
                const uint32_t row2 = lds_addr(&L.wx[8 * RS + ro]);
                const float4 sk = S.set[s ? 1 : 0][2];   // dz, 1 / lever arm, K, lever arm
                float xlo, xhi;
                bool all;   // no bracket, or one that overflowed: every pair
                bool on16 = false;
                if constexpr (H16) on16 = PL || L.h16[s ? 1 : 0].on;
                if (on16) {
                    if constexpr (H16) all = bracket16(L.h16[s ? 1 : 0], x0, tolc, xlo, xhi);
                } else if constexpr (PL) {
                    const float dz = sk.x;
                    float w0;
                    const float tc = slope_bracket(x0, x_mag, sk.y, tolc, w0);
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
                uint32_t ends[2] = {row2, row2};
                row_lower<NW>(ends, [xlo, xhi](int i, float v) { return i == 0 ? v < xlo : v <= xhi; });
                int lo = (int)(ends[0] - row2) >> 2, hi = (int)(ends[1] - row2) >> 2;
                if (all) { lo = 0; hi = L.win[s ? 11 : 8].y; }
                cnt[k] = item < n_items && hi > lo ? hi - lo : 0;
                code[k] = (NS == 2 ? (lane >> 5) << 13 : 0) | ((s ? 1 : 0) << 12) | (i0 << 6) | lo;
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
            // 32 pairs per pass: each item marks where its pairs begin among
            // them (or that they went on from before), and the last mark at or
            // before a lane is its item
            const uint32_t w0 = (uint32_t)code[0] | ((uint32_t)off0 << 16), w1 = (uint32_t)code[1] | ((uint32_t)off1 << 16);
            for (int f = 0; f < total_max; f += HALF) {
                L.mark[j] = 0;
                wave_sync();
                const int a0 = off0 - f, a1 = off1 - f;
                if (cnt[0] > 0 && a0 < HALF && a0 + cnt[0] > 0) L.mark[a0 > 0 ? a0 : 0] = (uint32_t)j;
                if (cnt[1] > 0 && a1 < HALF && a1 + cnt[1] > 0) L.mark[a1 > 0 ? a1 : 0] = (uint32_t)(HALF + j);
                wave_sync();
                uint32_t m = L.mark[j];
                wave_sync();
                m = umax(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x111, 0xF, 0xF, true));
                m = umax(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x112, 0xF, 0xF, true));
                m = umax(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x114, 0xF, 0xF, true));
                m = umax(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x118, 0xF, 0xF, true));
                m = umax(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x142, 0xA, 0xF, false));
                const int src = (lane & HALF) | (int)(m & (HALF - 1));
                const uint32_t v0 = (uint32_t)__shfl((int)w0, src), v1 = (uint32_t)__shfl((int)w1, src);
                const uint32_t w = m >= HALF ? v1 : v0;
                triplets(lane, f + j < total, (w & 0xffffu) + (uint32_t)(f + j) - (w >> 16), nA, nB, tolc, low_p, tx_in,
                         qop, x_mag);
            }
        }

        if constexpr (NS == 2) {
            // one pool of n_triplets for both sides: each list is cut where its
            // entries' ranks among both reach it
            const uint64_t mine = L.tk[j & (MT - 1)];
            const Half &O = S.h[lane < HALF ? 1 : 0];
            const int n_max = nA > nB ? nA : nB;
            int r = j;
            for (int i = 0; i < n_max; i += 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) r += O.tk[i + k] < mine ? 1 : 0;
            }
            const uint64_t keep = __ballot(j < (lane >= HALF ? nB : nA) && r < P->n_triplets);
            nA = __popc((uint32_t)keep);
            nB = __popc((uint32_t)(keep >> HALF));
        }

        int best_r = -1;    // this half's best candidate
        float best_Q = 0.0f;
        if (nA + nB > 0) {
            candidates(lane, nA, nB, T_uv);
            best_r = fits(lane, lane >= HALF ? nB : nA, T_uv, y_in, ty_in, best_Q);
        }
        bool mine = act;    // this half writes the slot
        if constexpr (NS == 2) {
            // the lower Q of the two sides, of equal ones the lower key
            const int other_r = __shfl_xor(best_r, HALF);
            const float other_Q = __shfl_xor(best_Q, HALF);
            const uint64_t key = best_r >= 0 ? L.tk[best_r] : ~0ull;
            const uint64_t other = __shfl_xor((unsigned long long)key, HALF);
            if (other_r < 0) mine = best_r >= 0 || lane < HALF;
            else mine = best_r >= 0 && (best_Q < other_Q || (best_Q == other_Q && key < other));
        }

        // ---- output ----
        if (!mine) return;
        const bool found = best_r >= 0;
        if (j == 0) {
            const float4 f0 = L.fit[0], f1 = L.fit[1];
            const float bfa = f0.x, bfb = f0.y, bfc = f0.z, bfy0 = f0.w, bfty = f1.x;
            const float uT = P->z_T - P->z_ref;
            const float txT = bfb + 2.0f * bfc * uT + 3.0f * bfc * dR * uT * uT;
            const float qo = paper ? (kick_s(txT, bfty) - kick_s(tx_in, ty_in)) / field_F(fc, txT - tx_in)
                                   : div_by(txT - tx_in, P->r_kick);
            st32(B.found, t, (uint8_t)(found ? 1 : 0));
            st32(B.nhits, t, (uint8_t)(found ? __float_as_int(f1.z) : 0));
            st32(B.a, t, found ? bfa : 0.0f);
            st32(B.b, t, found ? bfb : 0.0f);
            st32(B.c, t, found ? bfc : 0.0f);
            st32(B.y0, t, found ? bfy0 : 0.0f);
            st32(B.ty, t, found ? bfty : 0.0f);
            st32(B.qop, t, found ? qo : 0.0f);
            st32(B.Q, t, found ? f1.y : 0.0f);
        }
        if (j < NL) {
            const int h = found ? (int)L.ch[best_r][j] : -1;
            st32(B.hit_idx, t * NL + (uint32_t)j, h >= 0 ? first + h : -1);
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

    // The constants of binary16 seeding: lane s of a half computes those of set s.
    __device__ __forceinline__ void seeds16(int lane, float xc, float x_mag, float tolc) {
        const int j = lane & (HALF - 1);
        Half &L = S.h[lane >> 5];
        bool shared = true;   // lane s: set s's outer windows each share one z
        if constexpr (!PL) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int l = (k & 1 ? 3 : 0) + (k & 2 ? 8 : 0);   // 0, 3, 8, 11
                const int2 w = L.win[l];
                bool differ = false;
#pragma unroll
                for (int i = 0; i < NW / HALF; ++i) {
                    const int h = j + HALF * i;
                    if (h < w.y && __float_as_uint(ld32(B.hz, ebase + (uint32_t)(w.x + h))) !=
                                       __float_as_uint(ld32(B.hz, ebase + (uint32_t)w.x)))
                        differ = true;
                }
                const uint64_t bal = __ballot(differ);
                if ((uint32_t)(bal >> (lane & HALF)) != 0 && (j & 1) == (k & 1)) shared = false;
            }
        }
        const bool s = j & 1;
        const float c0 = __shfl(xc, (lane & HALF) + (s ? 3 : 0)), c1 = __shfl(xc, (lane & HALF) + (s ? 7 : 4)),
                    c2 = __shfl(xc, (lane & HALF) + (s ? 11 : 8));
        const float4 sa = S.set[s ? 1 : 0][1], sk = S.set[s ? 1 : 0][2];   // .., z0, z1; dz, .., K, lever arm
        float z0 = sa.z, dz = sk.x, lev = sk.w;
        bool on = true;
        if constexpr (!PL) {
            const int2 w0 = L.win[s ? 3 : 0], w2 = L.win[s ? 11 : 8];
            on = shared && w0.y > 0 && w2.y > 0;
            z0 = on ? ld32(B.hz, ebase + (uint32_t)w0.x) : 0.0f;
            dz = on ? ld32(B.hz, ebase + (uint32_t)w2.x) - z0 : 1.0f;
            lev = P->z_mag - z0;
        }
        const float K = sk.z;
        SeedSet16 h;
        h.c[0] = c0;
        h.c[1] = c1;
        h.c[2] = c2;
        h.on = on;
        h.hRZ = (_Float16)(1.0f / dz);
        h.hC02 = (_Float16)(c2 - c0);
        h.hE0 = (_Float16)(c0 - x_mag);
        h.hL0 = (_Float16)lev;
        h.hA = (_Float16)(sa.w - z0 * K);
        h.hKK = (_Float16)K;
        h.hB = (_Float16)(c0 * K - c1);
        h.pad = (_Float16)0.0f;
        h.pad2[0] = h.pad2[1] = 0;
        h.E0 = (float)h.hE0;
        h.C02 = (float)h.hC02;
        const float sl = (float)h.hRZ * (float)h.hL0;
        h.S = fabsf(sl);
        h.rs = 1.0f / sl;
        h.rL = 1.0f / fabsf((float)h.hL0);
        h.err = EPS16 * (6.0f * (float)(_Float16)P->magtol_max + 2.0f * h.S * fabsf(h.C02)) + 0.01f;
        if (j < 2) L.h16[j] = h;
    }
    static constexpr float EPS16 = 5.5e-4f;   // binary16's unit roundoff, 2^-11, and an eighth

    // The third-layer hits that can pass the binary16 magnet filter for first
    // hit x0; true: there is no bracket.  With m1 = E0 + x0 - c0 and s = RZ L0 of
    // the rounded constants, M = m1 + (x2 - c2 - (x0 - c0) + C02) s but for the
    // rounding of eight operations.  Each is off by 2^-11 of its result, and
    // where |M| < Tm, the largest tolerance, the results after the product with
    // L0 are bounded by b = Tm + |m1|, the terms before it by b / |s| and the
    // constants: together by 2^-11 (6 Tm + 6 |m1| + |x0 - c0| + 2 |s| (|C02| +
    // |x0 - c0|)), taken an eighth larger.
    __device__ __forceinline__ bool bracket16(const SeedSet16 &h, float x0, float tolc, float &xlo, float &xhi) const {
        const float x0r = x0 - h.c[0], m1 = h.E0 + x0r, am1 = fabsf(m1), ax0 = fabsf(x0r);
        const float tmax = (float)(_Float16)P->magtol_max, tmin = (float)(_Float16)P->magtol_min;
        const float txs = P->magtol_txscale > 0.0f ? (float)(_Float16)P->magtol_txscale : 0.0f;
        const float raw = (float)(_Float16)tolc + txs * ((tmax + am1) * h.rL);
        float tolb = raw + (2e-3f * fabsf(raw) + 1e-6f);
        if (tolb < tmin) tolb = tmin;
        if (tolb > tmax) tolb = tmax;
        const float W = tolb + h.err + EPS16 * (6.0f * am1 + ax0 + 2.0f * h.S * ax0);
        const float q = m1 * h.rs;
        const float e = h.c[2] + ((x0r - h.C02) - q);
        const float w0 = W * fabsf(h.rs);
        const float w = w0 + (0.05f + 1e-5f * (fabsf(e) + w0 + fabsf(q) + fabsf(h.c[2])));
        xlo = e - w;
        xhi = e + w;
        return !(fabsf(e) + w < 1e30f);
    }

    // Seed pair (x0, x2) in binary16: the filters, the closest middle hit (its
    // index in the row at row1: best) and its squared distance.  The operations
    // are Track's, in the same order.
    __device__ __forceinline__ bool triplet16(const SeedSet16 &h, bool in, float x0, float x2, uint32_t row1, float tolc,
                                              bool low_p, float tx_in, float qop, uint32_t &best, float &chi2) const {
        const _Float16 X0 = (_Float16)(x0 - h.c[0]);
        const _Float16 X2 = (_Float16)(x2 - h.c[2]);
        const _Float16 u = X2 - X0;
        const _Float16 v = u + h.hC02;
        const _Float16 t = v * h.hRZ;
        const _Float16 w1 = t - (_Float16)tx_in;
        const _Float16 w2 = w1 * (_Float16)qop;
        bool ok = in && !(low_p && !(w2 > (_Float16)0.0f));
        const _Float16 m1 = h.hE0 + X0;
        const _Float16 m2 = t * h.hL0;
        const _Float16 M = m1 + m2;
        const _Float16 r1 = (_Float16)P->magtol_txscale * habs(t);
        _Float16 tol = (_Float16)tolc + r1;
        const _Float16 tmin = (_Float16)P->magtol_min, tmax = (_Float16)P->magtol_max;
        if (tol < tmin) tol = tmin;
        if (tol > tmax) tol = tmax;
        if (!(habs(M) < tol)) ok = false;
        const _Float16 a1 = t * h.hA;
        const _Float16 a2 = X0 * h.hKK;
        const _Float16 a3 = a1 + a2;
        const _Float16 X1e = a3 + h.hB;
        const float c1 = h.c[1];
        // the row's binary16 values Y are sorted and +inf past the window's end
        uint32_t p[1] = {row1};
        row_lower<NW>(p, [c1, X1e](int, float x) { return (_Float16)(x - c1) < X1e; });
        auto D = [c1, X1e](uint32_t a) { return habs((_Float16)(lds_at(a) - c1) - X1e); };
        const uint32_t pm = p[0] > row1 ? p[0] - 4u : row1;
        const _Float16 d = D(p[0]), dl = D(pm);
        const bool left = p[0] > row1 && !(dl > d);
        uint32_t a = left ? pm : p[0];
        const _Float16 hb = left ? dl : d;
        const _Float16 c2h = hb * hb;
        chi2 = (float)c2h;
        ok = ok && c2h < (_Float16)P->T_triplet;
        // equal distances before the left neighbour: binary16 has many far from
        // the prediction, so only where the triplet passes (160,000 tracks 217
        // -> 187 us, 20 dense events 125 -> 73)
        if (ok && left)
            while (a > row1 && D(a - 4u) == dl) a -= 4u;
        best = (a - row1) >> 2;
        return ok;
    }

    // Up to 32 seed pairs per half (one per lane, in: the lane has one): the
    // doublet filters, the closest middle hit, the triplet cut, and the merge
    // of the accepted triplets into the half's top-n list.
    __device__ __forceinline__ void triplets(int lane, bool in, uint32_t e, int &nA, int &nB, float tolc, bool low_p,
                                             float tx_in, float qop, float x_mag) {
        const int j = lane & (HALF - 1);
        Half &L = S.h[lane >> 5];
        const int NT = P->n_triplets;
        const bool s = (e >> 12) & 1u;
        const int i0 = (int)((e >> 6) & 63u), i2 = (int)(e & 63u);
        const int ro = s ? 3 * RS : 0;
        const float x0 = L.wx[ro + (i0 & (NW - 1))], x2 = L.wx[8 * RS + ro + (i2 & (NW - 1))];
        bool ok, on16 = false;
        uint32_t best = 0;
        float chi2 = 0.0f;
        const uint32_t row1 = lds_addr(&L.wx[4 * RS + ro]);
        if constexpr (H16) {
            on16 = PL || L.h16[s ? 1 : 0].on;
            if (on16) ok = triplet16(L.h16[s ? 1 : 0], in, x0, x2, row1, tolc, low_p, tx_in, qop, best, chi2);
        }
        if (!on16) {
            const float4 sa = S.set[s ? 1 : 0][1], sk = S.set[s ? 1 : 0][2];   // .., z0, z1; dz, .., K, lever arm
            float z0 = sa.z, dz = sk.x, lev = sk.w;
            if constexpr (!PL) {
                z0 = in ? ld32(B.hz, ebase + (uint32_t)(L.win[s ? 3 : 0].x + i0)) : 0.0f;
                dz = (in ? ld32(B.hz, ebase + (uint32_t)(L.win[s ? 11 : 8].x + i2)) : 1.0f) - z0;
                lev = P->z_mag - z0;
            }
            const float txd = PL ? div_by(x2 - x0, S.rset[s ? 1 : 0][0].x) : (x2 - x0) / dz;
            ok = in && !(low_p && !((txd - tx_in) * qop > 0.0f));
            const float xm = x0 + txd * lev;
            float tol = tolc + P->magtol_txscale * fabsf(txd);
            if (tol < P->magtol_min) tol = P->magtol_min;
            if (tol > P->magtol_max) tol = P->magtol_max;
            if (!(fabsf(xm - x_mag) < tol)) ok = false;
            const float x1e = sa.w * txd + (x0 - txd * z0) * sk.z;
            uint32_t p1[1] = {row1};
            row_lower<NW>(p1, [x1e](int, float v) { return v < x1e; });
            float bd;
            best = (row_closest(row1, 0.0f, x1e, p1[0], bd) - row1) >> 2;
            chi2 = bd * bd;
            ok = ok && bd < INFINITY && chi2 < P->T_triplet;
        }
        const uint64_t key = ((uint64_t)__float_as_uint(chi2) << 32) | e;
        // a full list only admits keys below its last one
        ok = ok && key < L.tk[NT - 1];
        const uint64_t bal = __ballot(ok);
        if (bal == 0) return;

        // merge: an element's place is its rank among the kept and the new keys
        const uint32_t bal_a = (uint32_t)bal, bal_b = (uint32_t)(bal >> HALF);
        const uint32_t mine_bal = lane >= HALF ? bal_b : bal_a;
        const int nb_a = __popc(bal_a), nb_b = __popc(bal_b), nb_max = nb_a > nb_b ? nb_a : nb_b;
        const int nL = lane >= HALF ? nB : nA, nL_max = nA > nB ? nA : nB;
        // (the lists are read four keys at a time, past their ends ~0)
        const uint64_t old = L.tk[j & (MT - 1)];
        const int oh1 = L.th1[j & (MT - 1)];
        int r_new = 0, r_old = j;
        L.nk[j] = ~0ull;
        wave_sync();
        if (ok) L.nk[__popc(mine_bal & ((1u << j) - 1u))] = key;
        wave_sync();
        if (nL_max == 0) {
            for (int i = 0; i < nb_max; i += 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) r_new += L.nk[i + k] < key ? 1 : 0;
            }
        } else {
            for (int i = 0; i < nL_max; i += 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) r_new += L.tk[i + k] < key ? 1 : 0;
            }
            for (int i = 0; i < nb_max; i += 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint64_t v = L.nk[i + k];
                    r_new += v < key ? 1 : 0;
                    r_old += v < old ? 1 : 0;
                }
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
        nA = nA + nb_a < NT ? nA + nb_a : NT;
        nB = nB + nb_b < NT ? nB + nb_b : NT;
        wave_sync();
    }

    // Triplet x(z) models and the extension to the missing layers: four lanes
    // per candidate, sixteen candidates per pass, the first track's and then
    // the second's.  Lanes 0..2 of a quad take a station each: its seed hit, and
    // the searches of its three other layers side by side.  nA, nB: the tracks'
    // candidates.
    __device__ __forceinline__ void candidates(int lane, int nA, int nB, float T_uv_) {
        const int st = lane & 3, sq = st < 3 ? st : 0;
        for (int k0 = 0; k0 < nA + nB; k0 += WAVE / 4) {
            const int kk = k0 + (lane >> 2);
            const bool on = kk < nA + nB, second = kk >= nA;
            const int k = second ? kk - nA : kk, r = on ? k : 0;
            Half &L = S.h[second ? 1 : 0];
            const uint32_t rows = lds_addr(&L.wx[4 * sq * RS]);
            const float T_uv = second ? bcast_f(T_uv_, HALF) : bcast_f(T_uv_, 0);
            uint32_t eb = 0;
            if constexpr (!PL)
                eb = (uint32_t)(second ? __builtin_amdgcn_readlane((int)ebase, HALF) : __builtin_amdgcn_readlane((int)ebase, 0));
            const uint32_t id = (uint32_t)L.tk[r];
            const bool s = (id >> 12) & 1u;
            // (masked: a half without candidates reads within its rows)
            const int i0 = (int)((id >> 6) & 63u) & (NW - 1), i2 = (int)(id & 63u) & (NW - 1), i1 = L.th1[r] & (NW - 1);
            const int ro = s ? 3 * RS : 0;
            const float X0 = L.wx[ro + i0], X1 = L.wx[4 * RS + ro + i1], X2 = L.wx[8 * RS + ro + i2];
            float u0, g0, du01 = 0.0f, du12 = 0.0f, G01, dG = 0.0f;
            if constexpr (PL) {
                const float4 sm = S.set[s ? 1 : 0][0];
                u0 = sm.x; g0 = sm.y;
                G01 = S.set[s ? 1 : 0][1].x;
            } else {
                const float dR = P->dRatio;
                u0 = on ? ld32(B.hz, eb + (uint32_t)(L.win[s ? 3 : 0].x + i0)) - P->z_ref : 0.0f;
                const float u1 = on ? ld32(B.hz, eb + (uint32_t)(L.win[s ? 7 : 4].x + i1)) - P->z_ref : 0.0f;
                const float u2 = on ? ld32(B.hz, eb + (uint32_t)(L.win[s ? 11 : 8].x + i2)) - P->z_ref : 0.0f;
                g0 = g_of(u0, dR);
                const float g1 = g_of(u1, dR), g2 = g_of(u2, dR);
                du01 = u1 - u0;
                du12 = u2 - u1;
                const float G = (st == 0 ? g1 - g0 : g2 - g1) / (st == 0 ? du01 : du12);
                G01 = quad<0x00>(G);
                dG = quad<0x55>(G) - G01;
            }
            // lanes 0 and 1 divide for the two secant slopes
            float q, s01, s12, c;
            if constexpr (PL) {
                const double2 ra = S.rset[s ? 1 : 0][0], rb = S.rset[s ? 1 : 0][1];   // .., u1 - u0; u2 - u1, dG
                q = div_by(st == 0 ? X1 - X0 : X2 - X1, st == 0 ? ra.y : rb.x);
                s01 = quad<0x00>(q);
                s12 = quad<0x55>(q);
                c = div_by(s12 - s01, rb.y);
            } else {
                q = (st == 0 ? X1 - X0 : X2 - X1) / (st == 0 ? du01 : du12);
                s01 = quad<0x00>(q);
                s12 = quad<0x55>(q);
                c = (s12 - s01) / dG;
            }
            const float b = s01 - c * G01;
            const float a = X0 - b * u0 - c * g0;
            if (on && st == 0) {
                L.ca[k] = a;
                L.cb[k] = b;
                L.cc[k] = c;
            }
            // the station's x layer without the seed hit, then u and v
            const float4 y[3] = {L.lay[4 * sq + (s ? 0 : 3)], L.lay[4 * sq + 1], L.lay[4 * sq + 2]};
            const float xe[3] = {a + b * y[0].x + c * y[0].y, a + b * y[1].x + c * y[1].y, a + b * y[2].x + c * y[2].y};
            const float cc[3] = {0.0f, PL ? y[1].z : 0.0f, PL ? y[2].z : 0.0f};
            const uint32_t row[3] = {rows + (s ? 0u : 12u * RS), rows + 4u * RS, rows + 8u * RS};
            uint32_t p[3] = {row[0], row[1], row[2]}, hit[3];
            row_lower<NW>(p, [&](int i, float v) { return (i == 0 ? v : v + cc[i]) < xe[i]; });
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                float bd;
                uint32_t at;
                if (PL || i == 0) {
                    at = row_closest(row[i], cc[i], xe[i], p[i], bd);
                } else {
                    const float W = y[i].w + 1e-6f * fabsf(xe[i]);
                    // (a lane without a candidate has nothing to walk)
                    const uint32_t n4 = on ? 4u * (uint32_t)L.win[4 * sq + i].y : 0u;
                    at = row_closest_near(row[i], row[i] + n4, xe[i], W, on ? p[i] : row[i], bd);
                }
                const bool keep = bd < INFINITY && bd * bd < (i == 0 ? P->T_x : T_uv);
                hit[i] = keep ? (at - row[i]) >> 2 : 0xFFu;
            }
            // the station's four hit bytes; a seed hit is the first (set 0) or
            // last (set 1) layer of its station
            const uint32_t seed = (uint32_t)(st == 0 ? i0 : st == 1 ? i1 : i2);
            const uint32_t word = (s ? hit[0] | (seed << 24) : seed | (hit[0] << 24)) | (hit[1] << 8) | (hit[2] << 16);
            if (on && st < 3) L.chw[k][sq] = word;
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
    // Returns the half's best candidate (its fit is in fit[], its
    // quality in best_Q), or -1.
    __device__ __forceinline__ int fits(int lane, int nL, float T_uv, float y_in, float ty_in, float &best_Q) {
        const int j = lane & (HALF - 1);
        Half &L = S.h[lane >> 5];
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
        const int st = j & 3, sq = st < 3 ? st : 0;   // lane 3 holds no layers
        const float dR = P->dRatio;
        double r_dxy[2] = {1.0, 1.0};
        if constexpr (PL) {
            r_dxy[0] = P->r_dxdy[4 * sq + 1];
            r_dxy[1] = P->r_dxdy[4 * sq + 2];
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
            float rr[4], R0, R1, R2, sv[4], h[4], dxy[2];
            bool pres[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pres[i] = !(absent & (0x80u << (8 * i)));
                const int hit = (int)((word >> (8 * i)) & 0x7Fu);
                const bool st_layer = i == 1 || i == 2;
                float xm = 0.0f, u, gu;
                if constexpr (PL) {
                    const float4 y = L.lay[4 * sq + i];   // u, g, dxdy y, h
                    // (an absent hit reads within the row and is dropped)
                    xm = L.wx[(4 * sq + i) * RS + (hit & (NW - 1))];
                    if (st_layer) xm = xm + y.z;
                    u = y.x;
                    gu = y.y;
                    sv[i] = u * INV1024;
                    h[i] = y.w;
                } else {
                    u = sv[i] = h[i] = gu = 0.0f;
                    if (st_layer) dxy[i - 1] = 1.0f;
                    if (pres[i]) {
                        const uint32_t gi = ebase + (uint32_t)(L.win[4 * sq + i].x + hit);
                        const float x = ld32(B.hx, gi), z = ld32(B.hz, gi);
                        u = z - P->z_ref;
                        xm = x;
                        if (st_layer) {
                            dxy[i - 1] = ld32(B.hd, gi);
                            xm = x + dxy[i - 1] * (y_in + ty_in * (z - P->z_in));
                        }
                        sv[i] = u * INV1024;
                        h[i] = sv[i] * sv[i] * (1.0f + dR * u);
                        gu = g_of(u, dR);
                    }
                }
                const float m = xm - (a + b * u + c * gu);
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
                F.r_nx = Ft->r_nx;
                F.r_ny = Ft->r_ny;
            }
            {
                const float q1[4] = {sv[0] * rr[0], sv[1] * rr[1], sv[2] * rr[2], sv[3] * rr[3]};
                const float q2[4] = {h[0] * rr[0], h[1] * rr[1], h[2] * rr[2], h[3] * rr[3]};
                R0 = quad_sum(rr);
                R1 = quad_sum(q1);
                R2 = quad_sum(q2);
            }
            if constexpr (PL) F = *Ft;
            const bool ok_x = fabsf(F.det) > 0.0f;
            const float det_s = ok_x ? F.det : 1.0f;
            // lanes 0, 1 and 2 divide the numerators of da, db and dc
            const float A = R1 * F.S22 - F.S12 * R2, E = R1 * F.S12 - F.S11 * R2, G = F.S1 * R2 - R1 * F.S2;
            const float num_x = st == 0 ? R0 * F.m00 - F.S1 * A + F.S2 * E
                              : st == 1 ? F.S0 * A - R0 * F.m01 + F.S2 * G
                                        : F.S0 * (F.S11 * R2 - R1 * F.S12) - F.S1 * G + R0 * F.m02;
            const float q_x = PL ? div_by(num_x, F.r_det) : num_x / det_s;
            const float da = quad<0x00>(q_x), db = quad<0x55>(q_x), dc = quad<0xAA>(q_x);
            float chi[4], eta[2], eta_s[2];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool st_layer = i == 1 || i == 2;
                const float res = rr[i] - (da + db * sv[i] + dc * h[i]);
                const float q = PL && !st_layer ? div_by(res * res, P->r_Tx) : res * res / (st_layer ? T_uv : P->T_x);
                chi[i] = pres[i] ? q : 0.0f;
                if (st_layer) {
                    const float y = PL ? div_by(-res, r_dxy[i - 1]) : -res / dxy[i - 1];
                    eta[i - 1] = pres[i] ? y : 0.0f;
                    eta_s[i - 1] = sv[i] * eta[i - 1];
                }
            }
            const float Qx = quad_sum(chi), Y0 = quad_sum(eta), Y1 = quad_sum(eta_s);
            const bool ok_y = fabsf(F.D) > 0.0f;
            const float D_s = ok_y ? F.D : 1.0f;
            const float num_y = st == 0 ? Y0 * F.YS11 - F.YS1 * Y1 : F.YS0 * Y1 - F.YS1 * Y0;   // of dy0, dty
            const float q_y = PL ? div_by(num_y, F.r_D) : num_y / D_s;
            const float dy0 = quad<0x00>(q_y), dty = quad<0x55>(q_y);
            const float dslope = dty * INV1024;
            float chy[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float ry = eta[i] - (dy0 + dty * sv[i + 1]);
                const float q = div_by(ry * ry, P->r_Ty);
                chy[i] = pres[i + 1] ? q : 0.0f;
            }
            const float Qy = quad_sum(chy);
            const float q_q = div_by(st == 0 ? Qx : Qy, st == 0 ? F.r_nx : F.r_ny);
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
