// The body of k_flux: one lane's edge e, Gauss point g and layer lay, in a function with the kernel's
// parameters and a constant LAY (the wave's layer; -1: the lanes hold both).  It is included and not
// called: inlined from a function, its FP32 products are contracted into other sums, and a few obtuse
// cells amplify the mixed path's rounding.  That keeps the bits with one compiler; another may contract
// the sums otherwise, as their order is not written out.
    if (e >= m.E) return;
    const int64_t T = m.T, E = m.E;
    const int sc = m.escen ? (int)GKS_IX(m.escen[e], m.S) : 0;
    const R dt = (R)p.scal[2 * sc];
    // a scenario that has reached its end time takes zero-length steps: nothing to evolve (both
    // lanes of a Gauss-point pair belong to the same edge and leave together)
    if (p.scal[2 * sc] == 0.0) return;
    const R chi = (R)p.chi[sc], G = (R)p.G;
    const int32_t L = GKS_IX(m.eL[e], m.T), Rc = m.eR[e] >= 0 ? GKS_IX(m.eR[e], m.T) : m.eR[e],
                  sl = m.eslot[e];
    const int kL = GKS_IX(sl & 3, 3), kR = GKS_IX(sl >> 2, 3);
    const R *en = tab<R>(m.en), *egB = tab<R>(m.egB);
    const R nx = en[e], ny = en[E + e], tx = -ny, ty = nx;
    const double Bg = m.eBgp[g * E + e];
    const R gBx = egB[e], gBy = egB[E + e];
    const int hq = lay == 0 ? 1 : 0;   // own thickness in the record (eta1 / h2)
    const int mq = lay == 0 ? 2 : 0;   // own momenta in the record
    const int gv = lay == 0 ? 3 : 0;   // own variables' gradients start at paper component gv
    const int fv = lay == 0 ? 0 : 3;   // the other layer's height drives this layer's force
    const int ff = lay == 0 ? 1 : 0;   // modelled field index (0: eta1, 1: h2)
    // nonlinear weight of the force model
    const R rL = r0[ff * T + L], rR = Rc >= 0 ? r0[ff * T + Rc] : rL;
    const R wf0 = fmin(R(1), fmin(rL, rR));
    const R wf = (double)wf0 < W_ONE ? wf0 : R(1);
    // wet/dry: at an edge of this layer's front band (r0 of its own field 0 on either side) the
    // evolution is of first order: the sides' states alone, no slopes, no acceleration
    const bool order1 = WD && (r0[(1 - ff) * T + L] == R(0) || (Rc >= 0 && r0[(1 - ff) * T + Rc] == R(0)));
    SideL<R> side[2];
    double h64[2];
#pragma unroll
    for (int s = 0; s < 2; s++) {
        if (s == 1 && Rc < 0) break;
        const int64_t cell = s == 0 ? L : Rc;
        const int64_t at = s == 0 ? rec_at(T, cell, kL, g) : rec_at(T, cell, kR, 1 - g);
        const GpHead<R> *hp = rec.head + at;
        const R *rm = hp->q, *rg = rec.tail[at].g;
        double hh = hp->h[hq];
        const R ex = rg[2 * gv], ey = rg[2 * gv + 1];  // slope of h2, or of eta1
        R hx = ex, hy = ey;
        if (lay == 0) {  // eta1 -> h1 with the single-valued bottom at the Gauss point
            hh -= Bg;
            hx -= gBx;
            hy -= gBy;
        }
        h64[s] = hh;
        const R mx = rm[mq], my = rm[mq + 1];
        const R mxx = rg[2 + 2 * gv], mxy = rg[3 + 2 * gv];
        const R myx = rg[4 + 2 * gv], myy = rg[5 + 2 * gv];
        const R fx = rg[2 * fv], fy = rg[2 * fv + 1];
        // the plane gradient enters only where the weight is below 1 (it is not computed elsewhere)
        R dfx = fx, dfy = fy;
        if (wf < R(1)) {
            const R px1 = (R)gP1[(2 * ff) * T + cell], py1 = (R)gP1[(2 * ff + 1) * T + cell];
            dfx = wf * fx + (1 - wf) * px1;
            dfy = wf * fy + (1 - wf) * py1;
        }
        R ax, ay;
        if (lay == 0) {  // lower layer: upper-layer thickness (chi weighted); the bottom part -G gB
            ax = -chi * G * dfx;  // of its acceleration enters through bottom_moments
            ay = -chi * G * dfy;
        } else {         // upper layer: slope of the interface level
            ax = -G * dfx;
            ay = -G * dfy;
        }
        SideL<R> &q = side[s];
        // wet/dry: a side at or below h_dry is a vacuum (every term of it an exact zero)
        const bool vac = WD && !(hh > p.h_dry);
        if (vac) h64[s] = 0.0;
        const R h = vac ? R(0) : (R)hh, ih = vac ? R(0) : div_(R(1), h);
        q.h = h;
        q.ih = ih;
        q.U = (mx * nx + my * ny) * ih;
        q.V = (mx * tx + my * ty) * ih;
        q.hn = hx * nx + hy * ny;
        q.ht = hx * tx + hy * ty;
        q.en = ex * nx + ey * ny;
        q.et = ex * tx + ey * ty;
        const R dmn_x = mxx * nx + myx * ny, dmn_y = mxy * nx + myy * ny;  // grad (m . n)
        const R dmt_x = mxx * tx + myx * ty, dmt_y = mxy * tx + myy * ty;  // grad (m . t)
        q.mnn = dmn_x * nx + dmn_y * ny;
        q.mnt = dmn_x * tx + dmn_y * ty;
        q.mtn = dmt_x * nx + dmt_y * ny;
        q.mtt = dmt_x * tx + dmt_y * ty;
        q.pn = ax * nx + ay * ny;
        q.pt = ax * tx + ay * ty;
        if (order1) {
            q.hn = q.ht = q.en = q.et = R(0);
            q.mnn = q.mnt = q.mtn = q.mtt = R(0);
            q.pn = q.pt = R(0);
        }
    }
    if (Rc == -1) {  // wall: mirror image of the left side
        side[1] = side[0];
        side[1].U = -side[0].U;
        side[1].hn = -side[0].hn;
        side[1].en = -side[0].en;
        side[1].mnt = -side[0].mnt;
        side[1].mtn = -side[0].mtn;
        side[1].pn = -side[0].pn;
        h64[1] = h64[0];
    } else if (Rc < 0) {  // free boundary: every component extended evenly across the edge
        side[1] = side[0];
        side[1].hn = -side[0].hn;
        side[1].en = -side[0].en;
        side[1].mnn = -side[0].mnn;
        side[1].mtn = -side[0].mtn;
        side[1].pn = -side[0].pn;
        h64[1] = h64[0];
    }
    const double hbase = 0.5 * (h64[0] + h64[1]);
    // single-valued bottom slope in the local frame (zero normal part at walls by construction)
    const R gBn = (lay == 0 && !order1) ? gBx * nx + gBy * ny : R(0);
    const R gBt = (lay == 0 && !order1) ? gBx * tx + gBy * ty : R(0);
    R F0[3], Ft[3], Wb[3], Wbt[3];
    bool dry;
    if constexpr (LAY < 0)
        dry = gks_point<R, AM, WD>(side[0], side[1], hbase, gBn, gBt, G, (R)p.eps, (R)p.eps_num, dt, F0, Ft, Wb, Wbt,
                                   order1, p.h_dry);
    else
        dry = gks_point64<AM, WD, LAY == 0>(side[0], side[1], hbase, gBn, gBt, G, p.eps, p.eps_num, dt, F0, Ft, Wb, Wbt,
                                            order1, p.h_dry);
    if (Rc == -1) {  // no mass crosses a wall
        F0[0] = 0;
        Ft[0] = 0;
    }
    // FP64 hydrostatic pieces: interface thickness and 1/2 G hb^2, averaged over the two points
    // (both zero at a dry interface)
    const double hb = dry ? 0.0 : hbase + (double)Wb[0];
    double P = 0.5 * p.G * hb * hb, H = hb, Hc = hbase;
    P = 0.5 * (P + __shfl_xor(P, 1));
    H = 0.5 * (H + __shfl_xor(H, 1));
    // the layer coupling's Gauss-point thickness (Sec. 3.2, Eq. SWE-source-discretization), read as
    // the mean of the two sides' reconstructed values, and its rate, the mean of the sides' -div(h U)
    Hc = 0.5 * (Hc + __shfl_xor(Hc, 1));
    R Hct = R(-0.5) * ((side[0].mnn + side[0].mtt) + (side[1].mnn + side[1].mtt));
    Hct = R(0.5) * (Hct + __shfl_xor(Hct, 1));
    // the rest back to the global frame, then averaged over the two Gauss points
    R out[11];
    out[0] = F0[0];
    out[1] = F0[1] * nx + F0[2] * tx;
    out[2] = F0[1] * ny + F0[2] * ty;
    out[3] = Ft[0];
    out[4] = Ft[1] * nx + Ft[2] * tx;
    out[5] = Ft[1] * ny + Ft[2] * ty;
    R side_out[5];  // GM = 1: the right side's momenta and rates (the left side's go in out[6..10])
    if constexpr (GM == 1) {
        H = h64[0];
        double Hr = h64[1];
#pragma unroll
        for (int s = 0; s < 2; s++) {
            R r[3];
            side_rate(side[s], G, r);
            R *o5 = s == 0 ? out + 6 : side_out;
            const R mn = side[s].h * side[s].U, mt = side[s].h * side[s].V;
            o5[0] = mn * nx + mt * tx;
            o5[1] = mn * ny + mt * ty;
            o5[2] = r[0];
            o5[3] = r[1] * nx + r[2] * tx;
            o5[4] = r[1] * ny + r[2] * ty;
        }
        H = 0.5 * (H + __shfl_xor(H, 1));
        Hr = 0.5 * (Hr + __shfl_xor(Hr, 1));
#pragma unroll
        for (int i = 0; i < 5; i++) side_out[i] = R(0.5) * (side_out[i] + __shfl_xor(side_out[i], 1));
        if (g == 0) eoh[(int64_t)(lay == 0 ? 7 : 6) * E + e] = Hr;
    } else {
        out[6] = Wb[1] * nx + Wb[2] * tx;
        out[7] = Wb[1] * ny + Wb[2] * ty;
        out[8] = Wbt[0];
        out[9] = Wbt[1] * nx + Wbt[2] * tx;
        out[10] = Wbt[1] * ny + Wbt[2] * ty;
    }
#pragma unroll
    for (int i = 0; i < 11; i++) out[i] = R(0.5) * (out[i] + __shfl_xor(out[i], 1));
    const int o = lay == 0 ? 3 : 0;  // paper component offset of this layer
    if (g == 0) {
        if constexpr (STAGE == 0) eoh[(int64_t)(lay == 0 ? 1 : 0) * E + e] = P;
        eoh[(int64_t)(lay == 0 ? 3 : 2) * E + e] = H;
        eoh[(int64_t)(lay == 0 ? 5 : 4) * E + e] = Hc;
#pragma unroll
        for (int i = 0; i < 3; i++)
            if (STAGE == 0 || i == 0) eom[(int64_t)(o + i) * E + e] = out[i];      // F0
#pragma unroll
        for (int i = 0; i < 3; i++) eom[(int64_t)(6 + o + i) * E + e] = out[3 + i];  // Ft
    } else {
        const int mo = lay == 0 ? 2 : 0;
        if constexpr (STAGE == 0) {
            eom[(int64_t)(12 + mo) * E + e] = out[6];  // Wb momenta
            eom[(int64_t)(13 + mo) * E + e] = out[7];
        }
#pragma unroll
        for (int i = 0; i < 3; i++) eom[(int64_t)(16 + o + i) * E + e] = out[8 + i];  // Wbt
        eom[(int64_t)(lay == 0 ? 23 : 22) * E + e] = Hct;
        if constexpr (GM == 1) {
            if constexpr (STAGE == 0) {
                eom[(int64_t)(24 + mo) * E + e] = side_out[0];
                eom[(int64_t)(25 + mo) * E + e] = side_out[1];
            }
#pragma unroll
            for (int i = 0; i < 3; i++) eom[(int64_t)(28 + o + i) * E + e] = side_out[2 + i];
        }
    }
