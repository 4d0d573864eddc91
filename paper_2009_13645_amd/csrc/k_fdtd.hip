// k_fdtd.hip -- field kernels of the boosted-frame PIC step.
//
//  * Sweep / SweepVec: NSFD update of A_x, A_y, A_z and phi at interior
//    nodes (MITHRA 2.0 manual, sec. "FDTD for Wave Equation", eqs. NSFDtrick
//    and updateEquation; sec. "FDTD for Scalar Potential").  HBM-bound
//    15-point stencil: each thread owns one (i,j) column of a TX x TY tile
//    and marches along z with a register queue of psi^n(k-1..k+1); the
//    z-averaged value psi-bar of every column (plus a one-column halo ring)
//    goes through a double-buffered LDS plane, so psi^n is read from HBM
//    about once.  The source of the step (node-averaged edge current, or
//    rho) is read only on the x range that the last deposit may have touched
//    in each (plane, row).
//  * Mur: Mur absorbing boundaries (sec. "Boundary Truncation"), one thread
//    per boundary face node.  Faces use the printed first/second-order
//    updates with permuted axes; further workgroups clear the other source
//    set for the coming deposit.  Edges
//    and corners (MurEdge, mur_dev.hpp) follow in a later launch: they solve
//    the sum of the first-order conditions of their faces discretised at the
//    centre of the 2x2 (2x2x2) node stencil, reading the new face values (a
//    corner recomputes its edge neighbours).  Three time levels make all
//    reads race-free.
//  * VertexFields: E and B at vertices (sec. "Field Evaluation"):
//    E = -(A^{n+1} - A^n)/dt - grad phi, B = mean of curl A^n and curl A^{n+1}.
//  * StepFields: in a run of its own the Mur faces, the clearing, the vertex
//    fields, the power's partial sums and the plane's spectrum are one launch;
//    grouped steps launch Mur, then VertexPower.
#include "mithra_dev.hpp"
#include "mur_dev.hpp"
#include <algorithm>
#include <type_traits>

namespace mithra {

// ---------------------------------------------------------------------------
// K1: NSFD sweep
// ---------------------------------------------------------------------------

template <typename T>
__device__ inline T src_value(const RunDev &R, int comp, int set, int64_t c, int64_t back)
{
    // node-averaged edge current along comp, or rho; scaled to the update
    if (comp < 3) {
        const T *J = src_ptr<T>(R, set, comp);
        double s = (double)J[c] + (double)J[c - back];
        if (R.compensated) {
            const T *L = srclo_ptr<T>(R, set, comp);
            s += (double)L[c] + (double)L[c - back];
        }
        return (T)(R.sfac_A * 0.5 * s);
    }
    const T *Q = src_ptr<T>(R, set, 3);
    double s = (double)Q[c];
    if (R.compensated)
        s += (double)srclo_ptr<T>(R, set, 3)[c];
    return (T)(R.sfac_phi * s);
}

// FP32 sweeps use the difference form of the update,
//   psi^{n+1} = psi + [(psi - psi^{n-1}) + rx2 (d_xx psi + d_xx c)
//               + ry2 (d_yy psi + d_yy c) + rz2 d_zz psi + S],
//   c = psi-bar - psi = A ((psi_{k-1} - psi) + (psi_{k+1} - psi)),
// with every second difference formed from neighbour differences: for a
// smooth field those are exact in FP32, and psi enters once per step, so the
// rounding the leapfrog integrates is relative to the increment instead of
// to psi.  It is the same update as eq. updateEquation (its coefficients
// summed); FP64 sweeps keep the coefficient form.
template <typename T>
constexpr bool kDiffForm = sizeof(T) == 4;

template <typename T, int TX, int TY, int TZ>
struct Sweep {
    static constexpr int kThreads = TX * TY;
    static __device__ void run(const RunDev &R, Blk blk)
    {
        __shared__ T sb[2][TY + 2][TX + 2];
        // difference form: psi-bar - psi of the same node
        __shared__ T sbc[kDiffForm<T> ? 2 : 1][kDiffForm<T> ? TY + 2 : 1][TX + 2];

        // tiles start at node 0 so that every row load is 128-byte aligned; the
        // boundary columns load (they are the neighbours of the first interior
        // column) but are not updated
        const int ntx = (R.nx + TX - 1) / TX;
        const int nty = (R.ny + TY - 1) / TY;
        const int nch = (R.nz - 2 + TZ - 1) / TZ;
        int64_t lb = xcd_swizzle(blk.id, blk.n);
        const int tile_x = (int)(lb % ntx);
        lb /= ntx;
        const int tile_y = (int)(lb % nty);
        lb /= nty;
        const int chunk = (int)(lb % nch);
        const int comp = (int)(lb / nch);
        if (comp >= 4)
            return;  // grid larger than the tiling (never for the launchers here)

        const int64_t s = R.ctl->step;
        const int set_r = (int)(s & 1);

        const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
        const int i = tile_x * TX + lx;
        const int j = tile_y * TY + ly;
        const bool inb = (i < R.nx) && (j < R.ny);
        const bool valid = (i >= 1) && (j >= 1) && (i <= R.nx - 2) && (j <= R.ny - 2);
        const int ic = min(i, R.nx - 1), jc = min(j, R.ny - 1);
        const int64_t plane = (int64_t)R.nx * R.ny;
        const int64_t col = (int64_t)jc * R.nx + ic;

        // halo ring: left/right columns (TY each), bottom/top rows (TX each)
        const int H = 2 * (TX + TY);
        const int h = threadIdx.x;
        int hx = 0, hy = 0, hi_ = 0, hj_ = 0;
        bool hval = false;
        if (h < H) {
            if (h < TY) {
                hx = -1; hy = h;
            } else if (h < 2 * TY) {
                hx = TX; hy = h - TY;
            } else if (h < 2 * TY + TX) {
                hy = -1; hx = h - 2 * TY;
            } else {
                hy = TY; hx = h - 2 * TY - TX;
            }
            hi_ = tile_x * TX + hx;
            hj_ = tile_y * TY + hy;
            hval = (hi_ >= 0) && (hi_ < R.nx) && (hj_ >= 0) && (hj_ < R.ny);
        }
        const int64_t hcol = hval ? ((int64_t)hj_ * R.nx + hi_) : 0;

        const int kb = 1 + chunk * TZ;
        const int ke = min(kb + TZ, R.nz - 1);

        const T *cur = pot_ptr<T>(R, slot_cur(s), comp);
        const T *prev = pot_ptr<T>(R, slot_prev(s), comp);
        T *next = pot_ptr<T>(R, slot_next(s), comp);

        // source box of the set read now (expanded by one node on the high side:
        // a node average reaches the edge below it)
        const int *rlo = R.ctl->dep_lo[set_r];
        const int *rhi = R.ctl->dep_hi[set_r];
        const bool src_col = valid && i >= rlo[0] && i <= rhi[0] + 1 && j >= rlo[1] && j <= rhi[1] + 1;
        const int64_t back = comp == 0 ? 1 : (comp == 1 ? R.nx : plane);

        const T cA = (T)R.A, c1A = (T)(1.0 - 2.0 * R.A);
        const T a1 = (T)R.a1, a2 = (T)R.a2, a4 = (T)R.a4, a6 = (T)R.a6;
        const T rx2 = (T)R.rx2, ry2 = (T)R.ry2, rz2 = (T)R.rz2;

        T qm = 0, q0 = 0, qp = 0, hqm = 0, hq0 = 0, hqp = 0;
        if (inb) {
            qm = cur[(int64_t)(kb - 1) * plane + col];
            q0 = cur[(int64_t)kb * plane + col];
            qp = cur[(int64_t)(kb + 1) * plane + col];
        }
        if (hval) {
            hqm = cur[(int64_t)(kb - 1) * plane + hcol];
            hq0 = cur[(int64_t)kb * plane + hcol];
            hqp = cur[(int64_t)(kb + 1) * plane + hcol];
        }

        for (int k = kb; k < ke; ++k) {
            const int64_t c = (int64_t)k * plane + col;
            // issue the loads of this iteration before the barrier
            T pf = 0, hpf = 0;
            if (k + 1 < ke) {
                if (inb)
                    pf = cur[c + 2 * plane];
                if (hval)
                    hpf = cur[(int64_t)(k + 2) * plane + hcol];
            }
            T pm = 0, sv = 0;
            if (valid) {
                pm = prev[c];
                if (src_col && k >= rlo[2] && k <= rhi[2] + 1)
                    sv = src_value<T>(R, comp, set_r, c, back);
            }
            T(*buf)[TX + 2] = sb[k & 1];
            if constexpr (kDiffForm<T>) {
                T(*cbuf)[TX + 2] = sbc[k & 1];
                buf[ly + 1][lx + 1] = q0;
                cbuf[ly + 1][lx + 1] = cA * ((qm - q0) + (qp - q0));
                if (h < H) {
                    buf[hy + 1][hx + 1] = hq0;
                    cbuf[hy + 1][hx + 1] = cA * ((hqm - hq0) + (hqp - hq0));
                }
            } else {
                buf[ly + 1][lx + 1] = cA * (qm + qp) + c1A * q0;
                if (h < H)
                    buf[hy + 1][hx + 1] = cA * (hqm + hqp) + c1A * hq0;
            }
            __syncthreads();
            if (valid) {
                if constexpr (kDiffForm<T>) {
                    T(*cbuf)[TX + 2] = sbc[k & 1];
                    const T c0 = cbuf[ly + 1][lx + 1];
                    const T dxx = ((buf[ly + 1][lx] - q0) + (buf[ly + 1][lx + 2] - q0)) +
                                  ((cbuf[ly + 1][lx] - c0) + (cbuf[ly + 1][lx + 2] - c0));
                    const T dyy = ((buf[ly][lx + 1] - q0) + (buf[ly + 2][lx + 1] - q0)) +
                                  ((cbuf[ly][lx + 1] - c0) + (cbuf[ly + 2][lx + 1] - c0));
                    const T dzz = (qm - q0) + (qp - q0);
                    next[c] = q0 + ((q0 - pm) + rx2 * dxx + ry2 * dyy + rz2 * dzz + sv);
                } else {
                    T v = a1 * q0 + a2 * (buf[ly + 1][lx + 2] + buf[ly + 1][lx]) +
                          a4 * (buf[ly + 2][lx + 1] + buf[ly][lx + 1]) + a6 * (qp + qm) - pm + sv;
                    next[c] = v;
                }
            }
            qm = q0;
            q0 = qp;
            qp = pf;
            hqm = hq0;
            hq0 = hqp;
            hqp = hpf;
        }
    }
};

// Vectorised sweep: each thread owns V consecutive x-nodes (16-byte loads
// and stores), a tile is TXV*V nodes wide and TY rows high.  psi-bar of the
// tile plus a one-node halo ring goes through a double-buffered LDS plane
// whose interior starts on a 16-byte boundary; a thread reads its two outer
// x-neighbours and its y-neighbour vectors from LDS.  Needs nx % V == 0 so
// that every row starts aligned.
// Streaming (non-temporal) 16-byte accesses: data touched once per sweep
// (psi^{n-1} and psi^{n+1}) bypass cache retention so
// that the psi^n stencil planes stay in L2.
typedef unsigned int nt_u32x4 __attribute__((ext_vector_type(4)));

template <typename T, int V>
__device__ inline void vstore_nt(T *p, const Vec<T, V> &a)
{
    static_assert(sizeof(T) * V == 16, "16-byte vectors only");
    nt_u32x4 w;
    memcpy(&w, &a, 16);
    __builtin_nontemporal_store(w, reinterpret_cast<nt_u32x4 *>(p));
}

template <typename T, int V>
__device__ inline Vec<T, V> vload_nt(const T *p)
{
    static_assert(sizeof(T) * V == 16, "16-byte vectors only");
    const nt_u32x4 w = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4 *>(p));
    Vec<T, V> r;
    memcpy(&r, &w, 16);
    return r;
}

// Sources of one thread's V nodes on one plane: own edge/node values (a),
// the edge one step back along the component's axis (b, vector) or the
// left neighbour of the first node (lf, x component), with the two-sum low
// parts when compensated.
template <typename T, int V, bool LO>
struct PlaneSrc {
    Vec<T, V> pm, a, al, b, bl;
    T lf, lfl;
};

template <typename T, int V, int TXV, int TY, int TZ, bool LO>
struct SweepVec {
    static constexpr int kThreads = TXV * TY;
    static constexpr bool kCopyRun = true;  // see CopyRunOf
    static_assert(TZ % 4 == 0, "planes are processed four at a time");
    static constexpr int TW = TXV * V;                          // tile width in nodes
    static constexpr int ROW = ((V + TW + 1) + V - 1) / V * V;  // LDS row: pad(V-1), left halo, tile, right halo
    // source sums: FP64 for FP64 fields and for compensated FP32 (hi + lo)
    using ST = typename std::conditional<LO || sizeof(T) == 8, double, T>::type;
    struct Lds {
        __attribute__((aligned(16))) T sb[2][TY + 2][ROW];
        // difference form (FP32): psi-bar - psi of the same node
        __attribute__((aligned(16))) T sbc[kDiffForm<T> ? 2 : 1][kDiffForm<T> ? TY + 2 : 1][ROW];
        // psi^n at the two outermost nodes of each row end (x-face update)
        T rawe[2][TY + 2][4];
        // source row ranges of the tile's rows for the chunk's planes
        int2 sr[TZ][TY];
    };

    // OWN: a launch of a run of its own.  With tail it also carries the end of
    // the step before (SweepWithTail): the step number is then next_step, and
    // the deposit box, which that end writes, is not read.
    template <bool OWN = false>
    static __device__ __attribute__((always_inline)) void run(const RunDev &R, Blk blk, int tail = 0)
    {
        __shared__ Lds L;
        const int ntx = (R.nx + TW - 1) / TW;
        const int nty = (R.ny + TY - 1) / TY;
        const int nch = (R.nz - 2 + TZ - 1) / TZ;
        int64_t lb = xcd_swizzle(blk.id, blk.n);
        const int tile_x = (int)(lb % ntx);
        lb /= ntx;
        const int tile_y = (int)(lb % nty);
        lb /= nty;
        const int chunk = (int)(lb % nch);
        const int comp = (int)(lb / nch);
        if (comp >= (R.space_charge ? 4 : 3))
            return;  // grid larger than the tiling (never for the launchers here)
        const int64_t s = OWN && tail ? R.ctl->next_step : R.ctl->step;
        // the component is a compile-time constant inside the body, so the
        // source loads of the other components do not exist there
        switch (comp) {
        case 0: body<0, OWN>(R, L, tile_x, tile_y, chunk, s); break;
        case 1: body<1, OWN>(R, L, tile_x, tile_y, chunk, s); break;
        case 2: body<2, OWN>(R, L, tile_x, tile_y, chunk, s); break;
        default: body<3, OWN>(R, L, tile_x, tile_y, chunk, s); break;
        }
    }

    template <int COMP, bool OWN>
    static __device__ __attribute__((always_inline)) void body(const RunDev &R, Lds &L, int tile_x, int tile_y,
                                                               int chunk, int64_t s)
    {
        const int set_r = (int)(s & 1);

        const int lx = threadIdx.x % TXV, ly = threadIdx.x / TXV;
        const int i0 = tile_x * TW + lx * V;  // first node of this thread
        const int j = tile_y * TY + ly;
        const bool inb = (i0 < R.nx) && (j < R.ny);
        const bool work = inb && j >= 1 && j <= R.ny - 2;
        const int64_t plane = (int64_t)R.nx * R.ny;
        const int64_t col = inb ? ((int64_t)j * R.nx + i0) : 0;

        // Halo: bottom/top rows (TXV threads each), left/right columns (TY
        // threads each).  Every thread issues one aligned 16-byte halo load
        // per plane, so that no load is conditional: a column thread loads
        // the vector holding its node (element hsel), a thread without a
        // halo node reloads its own vector.
        const int t = threadIdx.x;
        int hrole = -1, hx = 0, hy = 0, hsel = 0;
        int64_t hv = col;
        bool hval = false;
        if (t < 2 * TXV) {
            hrole = 0;
            hx = (t % TXV) * V;
            hy = t < TXV ? -1 : TY;
            const int hi_ = tile_x * TW + hx, hj_ = tile_y * TY + hy;
            hval = hj_ >= 0 && hj_ < R.ny && hi_ < R.nx;
            if (hval)
                hv = (int64_t)hj_ * R.nx + hi_;
        } else if (t < 2 * TXV + 2 * TY) {
            hrole = 1;
            const int u = t - 2 * TXV;
            hy = u % TY;
            hx = u < TY ? -1 : TW;
            const int hi_ = tile_x * TW + hx, hj_ = tile_y * TY + hy;
            hval = hi_ >= 0 && hi_ < R.nx && hj_ < R.ny;
            hsel = hx < 0 ? V - 1 : 0;
            if (hval)
                hv = (int64_t)hj_ * R.nx + hi_ - hsel;
        }

        const int kb = 1 + chunk * TZ;
        const int ke = min(kb + TZ, R.nz - 1);
        const T *cur = pot_ptr<T>(R, slot_cur(s), COMP);
        const T *prev = pot_ptr<T>(R, slot_prev(s), COMP);
        T *next = pot_ptr<T>(R, slot_next(s), COMP);

        // the source row ranges of the set for the tile's rows and the
        // chunk's planes, through LDS (rows and planes clamped into the grid;
        // a clamped entry is never used for a stored node)
        {
            const int32_t *srl = R.srow_lo + (size_t)set_r * R.nz * R.ny;
            const int32_t *srh = R.srow_hi + (size_t)set_r * R.nz * R.ny;
            for (int e = threadIdx.x; e < TZ * TY; e += kThreads) {
                const int pz = e / TY, py = e - pz * TY;
                const int64_t row = (int64_t)min(kb + pz, R.nz - 1) * R.ny + min(tile_y * TY + py, R.ny - 1);
                L.sr[pz][py] = make_int2(srl[row], srh[row]);
            }
            __syncthreads();
        }
        // grouped: a column outside the deposit box has no sources
        bool src = work;
        if constexpr (!OWN) {
            const int *rlo = R.ctl->dep_lo[set_r], *rhi = R.ctl->dep_hi[set_r];
            src = src && i0 + V - 1 >= rlo[0] && i0 <= rhi[0] + 1 && j >= rlo[1] && j <= rhi[1] + 1;
        }
        const T *J = src_ptr<T>(R, set_r, COMP);
        const T *Jl = LO ? srclo_ptr<T>(R, set_r, COMP) : nullptr;
        const ST sfac = (ST)(COMP < 3 ? 0.5 * R.sfac_A : R.sfac_phi);

        const T cA = (T)R.A, c1A = (T)(1.0 - 2.0 * R.A);
        const T a1 = (T)R.a1, a2 = (T)R.a2, a4 = (T)R.a4, a6 = (T)R.a6;
        const T rx2 = (T)R.rx2, ry2 = (T)R.ry2, rz2 = (T)R.rz2;
        const int kmax = R.nz - 1;

        // psi^n of plane kk (own vector and halo vector); every plane index
        // is clamped into the array, so the loads need no guard
        auto load_cur = [&](int kk, Vec<T, V> &q, Vec<T, V> &h) {
            const int64_t o = (int64_t)min(kk, kmax) * plane;
            q = vload<T, V>(cur + o + col);
            h = vload<T, V>(cur + o + hv);
        };
        // psi^{n-1} and the sources of plane kk (kk <= nz - 1).  Outside the
        // row's source range the loads read node 0, which no deposit reaches
        // and which therefore holds zero; the z component's back edge is the
        // previous plane's own edge, carried in registers.
        auto fetch = [&](int kk, const PlaneSrc<T, V, LO> &prv, PlaneSrc<T, V, LO> &r) {
            const int64_t c = (int64_t)kk * plane + col;
            r.pm = vload_nt<T, V>(prev + c);
            // planes at or beyond ke are not stored: no source needed
            const int2 rg = L.sr[min(kk - kb, TZ - 1)][ly];
            const bool in = src && kk < ke && i0 + V - 1 >= rg.x && i0 <= rg.y;
            const int64_t ca = in ? c : 0;
            r.a = vload<T, V>(J + ca);
            if constexpr (LO)
                r.al = vload<T, V>(Jl + ca);
            if constexpr (COMP == 0) {
                const int64_t cl = in ? c - 1 : 0;
                r.lf = J[cl];
                if constexpr (LO)
                    r.lfl = Jl[cl];
            } else if constexpr (COMP == 1) {
                const int64_t cb = in ? c - R.nx : 0;
                r.b = vload<T, V>(J + cb);
                if constexpr (LO)
                    r.bl = vload<T, V>(Jl + cb);
            } else if constexpr (COMP == 2) {
                if (kk > kb) {
                    r.b = prv.a;
                    if constexpr (LO)
                        r.bl = prv.al;
                } else {
                    const int64_t cb = in ? c - plane : 0;
                    r.b = vload<T, V>(J + cb);
                    if constexpr (LO)
                        r.bl = vload<T, V>(Jl + cb);
                }
            }
        };

        // Plane k from the psi^n planes k-1, k, k+1 (qm, q0, qp; halo hm,
        // h0, hp) and the psi^{n-1} / source plane ps; the loads of plane
        // k+2 (pf, hpf) and of plane k+1 (pn) are issued first.  The caller
        // rotates the roles of the variables instead of copying them, so a
        // prefetch stays in flight across planes.  Planes at or beyond ke
        // (only in a chunk's last group of four) are computed and not stored.
        auto plane_step = [&](int k, const Vec<T, V> &qm, const Vec<T, V> &q0, const Vec<T, V> &qp, Vec<T, V> &pf,
                              const Vec<T, V> &hm, const Vec<T, V> &h0, const Vec<T, V> &hp, Vec<T, V> &hpf,
                              const PlaneSrc<T, V, LO> &ps, PlaneSrc<T, V, LO> &pn) {
            const int64_t c = (int64_t)k * plane + col;
            load_cur(k + 2, pf, hpf);
            fetch(min(k + 1, kmax), ps, pn);
            ST sv[V];
            if constexpr (COMP == 3) {
                for (int e = 0; e < V; ++e)
                    sv[e] = (ST)ps.a.v[e] + (LO ? (ST)ps.al.v[e] : (ST)0);
            } else if constexpr (COMP == 0) {
                ST left = (ST)ps.lf + (LO ? (ST)ps.lfl : (ST)0);
                for (int e = 0; e < V; ++e) {
                    const ST own = (ST)ps.a.v[e] + (LO ? (ST)ps.al.v[e] : (ST)0);
                    sv[e] = own + left;
                    left = own;
                }
            } else {
                for (int e = 0; e < V; ++e)
                    sv[e] = LO ? ((ST)ps.a.v[e] + (ST)ps.al.v[e]) + ((ST)ps.b.v[e] + (ST)ps.bl.v[e])
                               : (ST)ps.a.v[e] + (ST)ps.b.v[e];
            }
            T(*buf)[ROW] = L.sb[k & 1];
            // a column thread's halo node is element hsel of its vector
            const bool hl = hsel != 0;
            const T h0s = hl ? h0.v[V - 1] : h0.v[0], hms = hl ? hm.v[V - 1] : hm.v[0], hps = hl ? hp.v[V - 1] : hp.v[0];
            Vec<T, V> bar;  // psi-bar, or (difference form) psi-bar - psi
            if constexpr (kDiffForm<T>) {
                T(*cbuf)[ROW] = L.sbc[k & 1];
                for (int e = 0; e < V; ++e)
                    bar.v[e] = cA * ((qm.v[e] - q0.v[e]) + (qp.v[e] - q0.v[e]));
                vstore<T, V>(&buf[ly + 1][V + lx * V], q0);
                vstore<T, V>(&cbuf[ly + 1][V + lx * V], bar);
                if (hrole == 0) {
                    Vec<T, V> hb;
                    for (int e = 0; e < V; ++e)
                        hb.v[e] = cA * ((hm.v[e] - h0.v[e]) + (hp.v[e] - h0.v[e]));
                    vstore<T, V>(&buf[hy + 1][V + hx], h0);
                    vstore<T, V>(&cbuf[hy + 1][V + hx], hb);
                } else if (hrole == 1) {
                    buf[hy + 1][V + hx] = h0s;
                    cbuf[hy + 1][V + hx] = cA * ((hms - h0s) + (hps - h0s));
                }
            } else {
                for (int e = 0; e < V; ++e)
                    bar.v[e] = cA * (qm.v[e] + qp.v[e]) + c1A * q0.v[e];
                vstore<T, V>(&buf[ly + 1][V + lx * V], bar);
                if (hrole == 0) {
                    Vec<T, V> hb;
                    for (int e = 0; e < V; ++e)
                        hb.v[e] = cA * (hm.v[e] + hp.v[e]) + c1A * h0.v[e];
                    vstore<T, V>(&buf[hy + 1][V + hx], hb);
                } else if (hrole == 1) {
                    buf[hy + 1][V + hx] = cA * (hms + hps) + c1A * h0s;
                }
            }
            {
                T(*raw)[4] = L.rawe[k & 1];
                if (inb && i0 == 0) {
                    raw[ly + 1][0] = q0.v[0];
                    raw[ly + 1][1] = q0.v[1];
                }
                if (inb && i0 + V == R.nx) {
                    raw[ly + 1][2] = q0.v[V - 2];
                    raw[ly + 1][3] = q0.v[V - 1];
                }
                if (hrole == 0 && hval) {
                    const int hi_ = tile_x * TW + hx;
                    if (hi_ == 0) {
                        raw[hy + 1][0] = h0.v[0];
                        raw[hy + 1][1] = h0.v[1];
                    }
                    if (hi_ + V == R.nx) {
                        raw[hy + 1][2] = h0.v[V - 2];
                        raw[hy + 1][3] = h0.v[V - 1];
                    }
                }
            }
            __syncthreads();
            if (work && k < ke) {
                const T left = buf[ly + 1][V + lx * V - 1];
                const T right = buf[ly + 1][V + lx * V + V];
                const Vec<T, V> dn = vload<T, V>(&buf[ly][V + lx * V]);
                const Vec<T, V> up = vload<T, V>(&buf[ly + 2][V + lx * V]);
                Vec<T, V> out;
                if constexpr (kDiffForm<T>) {
                    T(*cbuf)[ROW] = L.sbc[k & 1];
                    const T cleft = cbuf[ly + 1][V + lx * V - 1];
                    const T cright = cbuf[ly + 1][V + lx * V + V];
                    const Vec<T, V> cdn = vload<T, V>(&cbuf[ly][V + lx * V]);
                    const Vec<T, V> cup = vload<T, V>(&cbuf[ly + 2][V + lx * V]);
                    for (int e = 0; e < V; ++e) {
                        const T p0 = q0.v[e], c0 = bar.v[e];
                        const T ql = e == 0 ? left : q0.v[e - 1], qr = e == V - 1 ? right : q0.v[e + 1];
                        const T cl = e == 0 ? cleft : bar.v[e - 1], cr = e == V - 1 ? cright : bar.v[e + 1];
                        const T dxx = ((ql - p0) + (qr - p0)) + ((cl - c0) + (cr - c0));
                        const T dyy = ((dn.v[e] - p0) + (up.v[e] - p0)) + ((cdn.v[e] - c0) + (cup.v[e] - c0));
                        const T dzz = (qm.v[e] - p0) + (qp.v[e] - p0);
                        out.v[e] = p0 + ((p0 - ps.pm.v[e]) + rx2 * dxx + ry2 * dyy + rz2 * dzz + (T)(sfac * sv[e]));
                    }
                } else {
                    for (int e = 0; e < V; ++e) {
                        const T xl = e == 0 ? left : bar.v[e - 1];
                        const T xr = e == V - 1 ? right : bar.v[e + 1];
                        out.v[e] = a1 * q0.v[e] + a2 * (xl + xr) + a4 * (dn.v[e] + up.v[e]) +
                                   a6 * (qp.v[e] + qm.v[e]) - ps.pm.v[e] + (T)(sfac * sv[e]);
                    }
                }
                // the x-face nodes of the row: Mur update (faces of the x
                // axis, transverse y and z), from this thread's own columns,
                // the neighbouring rows' values in LDS and the new inner
                // value.  When the Mur kernel also updates the x faces (a
                // scalar shape is the run's own), it runs after this kernel
                // and its values replace these.
                if (i0 == 0 || i0 + V == R.nx) {
                    const T(*raw)[4] = L.rawe[k & 1];
                    for (int side = 0; side < 2; ++side) {
                        if ((side == 0 && i0 != 0) || (side == 1 && i0 + V != R.nx))
                            continue;
                        const int eb = side == 0 ? 0 : V - 1, ei = side == 0 ? 1 : V - 2;
                        const int ro = side == 0 ? 0 : 2;
                        const int rb = side == 0 ? ro : ro + 1, ri = side == 0 ? ro + 1 : ro;
                        const Vec<T, V> &pm = ps.pm;
                        double v = R.mur_be0[0] * ((double)pm.v[eb] + (double)out.v[ei]) - (double)pm.v[ei];
                        if (R.order == 1) {
                            v += R.mur_be1[0] * ((double)q0.v[eb] + (double)q0.v[ei]);
                        } else {
                            v += R.mur_g1[0] * ((double)q0.v[eb] + (double)q0.v[ei]);
                            const double s1 = ((double)raw[ly][rb] + (double)raw[ly][ri]) +
                                              ((double)raw[ly + 2][rb] + (double)raw[ly + 2][ri]);
                            const double s2 = ((double)qm.v[eb] + (double)qm.v[ei]) + ((double)qp.v[eb] + (double)qp.v[ei]);
                            v += R.mur_ga[0] * s1;
                            v += R.mur_gb[0] * s2;
                        }
                        out.v[eb] = (T)v;
                    }
                }
                vstore_nt<T, V>(next + c, out);
            }
        };

        Vec<T, V> qm, q0, qp, pf, hm, h0, hp, hpf;
        load_cur(kb - 1, qm, hm);
        load_cur(kb, q0, h0);
        load_cur(kb + 1, qp, hp);
        PlaneSrc<T, V, LO> ps{}, pn{};
        fetch(kb, pn, ps);
        // four planes per iteration, the variables' roles rotating by one
        // plane each time (a period of four for the psi^n queues, two for
        // the psi^{n-1} / source planes); the last group of a chunk may run
        // up to three planes past ke, computed and not stored
        for (int k = kb; k < ke; k += 4) {
            plane_step(k, qm, q0, qp, pf, hm, h0, hp, hpf, ps, pn);
            plane_step(k + 1, q0, qp, pf, qm, h0, hp, hpf, hm, pn, ps);
            plane_step(k + 2, qp, pf, qm, q0, hp, hpf, hm, h0, ps, pn);
            plane_step(k + 3, pf, qm, q0, qp, hpf, hm, h0, hp, pn, ps);
        }
    }
};

// A sweep of a run of its own that, with `tail`, also ends the step before
// (BoxReduceEndStep, in the first workgroup): a launch of 4.6 us less a step,
// 72 x 56 x 136 nodes FP64 56 -> 53 us, 128 x 128 x 1024 FP32 373 -> 370.  Nothing that
// the end of a step writes is read by the sweep: it takes its own step number
// (next_step) and the source rows, not the deposit box.
template <class S>
struct SweepWithTail {
    static constexpr int kThreads = S::kThreads;
    static __device__ void run(const RunDev &R, Blk blk, int tail)
    {
        if (tail && blk.id == 0) {
            BoxReduceEndStep::run(R, Blk{0, 1});
            return;
        }
        S::template run<true>(R, Blk{blk.id - tail, blk.n - tail}, tail);
    }
};

// ---------------------------------------------------------------------------
// K2: Mur boundaries
// ---------------------------------------------------------------------------

// r / d for 0 <= r < half (r = row * d + column of a face): multiply-high
// when exact, else 64-bit division
__device__ inline uint32_t face_div(int64_t r, int64_t half, int d)
{
    if ((uint64_t)half * (uint64_t)d < (1ull << 32))
        return fdiv((uint32_t)r, fast_div((uint32_t)d));
    return (uint32_t)(r / d);
}

// Is node (i, j, k) a corner of an active cell whose sort tile is marked with
// a step of s - back .. s?  The push of step s-1 (or the load) marks the tiles
// of the cells its particles end in with s; a node's cells are i-1..i on each
// axis, within the active range 1..n-3.  The eight marks load without a branch
// between them.
__device__ inline bool node_marked(const RunDev &R, int64_t s, uint32_t back, int i, int j, int k)
{
    const uint32_t now = (uint32_t)s;
    uint32_t x[2], y[2], z[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        x[a] = fdiv((uint32_t)min(max(i - 1 + a, 1), R.nx - 3), R.tdiv[0]);
        y[a] = fdiv((uint32_t)min(max(j - 1 + a, 1), R.ny - 3), R.tdiv[1]);
        z[a] = fdiv((uint32_t)min(max(k - 1 + a, 1), R.nz - 3), R.tdiv[2]);
    }
    bool any = false;
#pragma unroll
    for (int a = 0; a < 8; ++a)
        any |= now - R.tile_flag[((int64_t)z[a >> 2] * R.ntile[1] + y[(a >> 1) & 1]) * R.ntile[0] + x[a & 1]] <= back;
    return any;
}

// Node t of a box, x fastest; by multiply-high when that is exact
// (t * max(ex, ey) < 2^32).
struct BoxNodes {
    int l0, l1, l2;
    int64_t ex, ey, tot;
    FastDiv fx, fy;
    bool fast;
    __device__ BoxNodes(int l0, int l1, int l2, int64_t ex, int64_t ey, int64_t ez)
        : l0(l0), l1(l1), l2(l2), ex(ex), ey(ey), tot(ex * ey * ez), fx(fast_div((uint32_t)ex)),
          fy(fast_div((uint32_t)ey)), fast((uint64_t)tot * (uint64_t)(ex > ey ? ex : ey) < (1ull << 32))
    {
    }
    __device__ void node(int64_t t, int &i, int &j, int &k) const
    {
        if (fast) {
            const uint32_t t32 = (uint32_t)t, row = fdiv(t32, fx);
            const uint32_t kk = fdiv(row, fy);
            i = l0 + (int)(t32 - row * (uint32_t)ex);
            j = l1 + (int)(row - kk * (uint32_t)ey);
            k = l2 + (int)kk;
        } else {
            i = l0 + (int)(t % ex);
            j = l1 + (int)((t / ex) % ey);
            k = l2 + (int)(t / (ex * ey));
        }
    }
};

// The source set that this step's deposit accumulates into is zeroed where
// its previous deposit, by the push of step s-2, may lie.  The set was last
// read by the previous step's sweep, and the deposit runs after this kernel.
// A deposit lies at the corners of the active cells in which that push began
// and ended a particle's move, within the set's node box.  The tiles of those
// cells carry a mark of s-2 (where moves began; set before that push), s-1
// (where they ended) or, renewed since, s.  Tiles never marked hold -1, so at
// step 1, whose set the load deposits into without marking where its moves
// begin, every node of the box counts.
// Bound by its writes, which also push the sweep's planes out of the last-level
// cache: of the 4.0 million nodes in example 1's box (64 x 64 x 2800 FP64) the
// marked tiles hold a third, and zeroing the whole box (rows of it, one
// wavefront each) took 485 us a step, this 454 (the sweep 200 -> 179, this
// launch 131 -> 123); 128 x 128 x 1024 FP32 367 -> 357.
// Boxes of few bytes are zeroed whole: there the caches take the writes, and
// looking up the marks costs more (5 MB at 64 x 64 x 384 FP32: 84.5 us a step
// zeroed whole, 85.9 by marks; 16 to 30 MB at 128 x 128 x 1024 FP32: 357.4
// against 354.7 by marks).  Particles over the whole grid leave little to skip
// and the marks' loads cost up to 3 % of the step: 128 x 128 x 128 FP64 with 1e5
// particles 193.7 whole and 199.7 by marks, 128 x 128 x 256 with 2e6 1440 and
// 1448, 64 x 64 x 1024 with 2e6 1136 and 1142.
constexpr int64_t kZeroAll = 8 << 20;

template <typename T>
__device__ inline void clear_next_sources(const RunDev &R, int64_t b, int64_t nb)
{
    const int64_t s = R.ctl->step;
    const int set_c = (int)((s + 1) & 1);
    const int *lo = R.ctl->dep_lo[set_c];
    const int *hi = R.ctl->dep_hi[set_c];
    const int l0 = lo[0], l1 = lo[1], l2 = lo[2];
    const int ex = hi[0] - l0 + 1, ey = hi[1] - l1 + 1, ez = hi[2] - l2 + 1;
    if (ex <= 0 || ey <= 0 || ez <= 0)
        return;
    const int64_t first = b * blockDim.x + threadIdx.x, step = nb * blockDim.x;
    // the set's source row ranges, on the rows the deposit's boxes may have
    // grown them to (one more node along y and z)
    {
        int32_t *slo = R.srow_lo + (size_t)set_c * R.nz * R.ny;
        int32_t *shi = R.srow_hi + (size_t)set_c * R.nz * R.ny;
        const int ry = ey + 1, nr = ry * (ez + 1);
        for (int64_t r = first; r < nr; r += step) {
            const int64_t row = (int64_t)(l2 + (int)(r / ry)) * R.ny + (l1 + (int)(r % ry));
            slo[row] = 0x7f7f7f7f;
            shi[row] = -1;
        }
    }
    const BoxNodes box(l0, l1, l2, ex, ey, ez);
    const bool all = box.tot * 4 * (int64_t)sizeof(T) <= kZeroAll;
    int i, j, k;
    auto marked = [&](int64_t t) {
        box.node(t, i, j, k);
        return all || node_marked(R, s, 2, i, j, k);
    };
    int64_t t = first;
    bool next = t < box.tot && marked(t);
    while (t < box.tot) {
        const bool now = next;
        const int64_t at = nid(R, i, j, k);
        t += step;  // the next node's marks load before this node's stores
        next = t < box.tot && marked(t);
        if (!now)
            continue;
#pragma unroll
        for (int comp = 0; comp < 4; ++comp) {
            src_ptr<T>(R, set_c, comp)[at] = (T)0;
            if (R.compensated)
                srclo_ptr<T>(R, set_c, comp)[at] = (T)0;
        }
    }
}

// workgroups that clear the next source set, after the Mur workgroups
static __host__ __device__ inline int64_t clear_blocks_of(int ny, int nz)
{
    const int64_t r = (int64_t)ny * nz / 64;
    return r < 8 ? 8 : (r > 2048 ? 2048 : r);
}

// Face workgroups (per component) plus the source-clearing workgroups.
__host__ __device__ inline int64_t mur_blocks_of(const RunDev &R)
{
    const int64_t nx = R.nx, ny = R.ny, nz = R.nz;
    const int64_t nodes = 2 * (nx - 2) * (ny - 2) + 2 * (nx - 2) * (nz - 2) + (R.xface_fused ? 0 : 2 * (ny - 2) * (nz - 2));
    return ((nodes + 255) / 256) * (R.space_charge ? 4 : 3) + clear_blocks_of(R.ny, R.nz);
}

// The n+1 value of face node c of axis ax from the levels n-1 (pm) and n
// (p0), the new value npq of q, its neighbour inside, and the strides s1, s2
// of the axes ax + 1 and ax + 2.
template <typename T>
__device__ inline T mur_face(const RunDev &R, int ax, const T *pm, const T *p0, double npq, int64_t c, int64_t q,
                             int64_t s1, int64_t s2)
{
    // coefficients by selects (no array indexed at run time)
    auto co = [ax](const double (&a)[3]) { return ax == 0 ? a[0] : (ax == 1 ? a[1] : a[2]); };
    double v = co(R.mur_be0) * ((double)pm[c] + npq) - (double)pm[q];
    if (R.order == 1) {
        v += co(R.mur_be1) * ((double)p0[c] + (double)p0[q]);
    } else {
        v += co(R.mur_g1) * ((double)p0[c] + (double)p0[q]);
        const double a1 = ((double)p0[c - s1] + (double)p0[q - s1]) + ((double)p0[c + s1] + (double)p0[q + s1]);
        const double a2 = ((double)p0[c - s2] + (double)p0[q - s2]) + ((double)p0[c + s2] + (double)p0[q + s2]);
        v = v + co(R.mur_ga) * a1 + co(R.mur_gb) * a2;
    }
    return (T)v;
}

// Face nodes of the boundary, one thread each (per component): z faces, y
// faces, and the x faces unless the vector sweep updated them, with direct
// strides, laid out x fastest so that their accesses coalesce.  The
// workgroups after the boundary ones clear the next source set
// (clear_next_sources).  Edge and corner nodes follow in MurEdge.
template <typename T>
struct Mur {
    static constexpr int kThreads = 256;
    static __device__ void run(const RunDev &R, Blk blk)
    {
        const int nx = R.nx, ny = R.ny, nz = R.nz;
        const int64_t fz = 2LL * (nx - 2) * (ny - 2);
        const int64_t fy = 2LL * (nx - 2) * (nz - 2);
        const int64_t fx = R.xface_fused ? 0 : 2LL * (ny - 2) * (nz - 2);
        const int64_t nb = fz + fy + fx;
        // ceil(nb / 256) workgroups per component (component uniform per
        // workgroup), then the workgroups that clear the next source set
        const int64_t bpc = (nb + 255) / 256;
        const int64_t nmur = bpc * (R.space_charge ? 4 : 3);
        if (blk.id >= nmur) {
            clear_next_sources<T>(R, blk.id - nmur, blk.n - nmur);
            return;
        }
        const int comp = (int)(blk.id / bpc);
        int64_t r = (blk.id - (int64_t)comp * bpc) * blockDim.x + threadIdx.x;
        if (r >= nb)
            return;
        const int64_t s = R.ctl->step;
        const T *pm = pot_ptr<T>(R, slot_prev(s), comp);
        const T *p0 = pot_ptr<T>(R, slot_cur(s), comp);
        T *pp = pot_ptr<T>(R, slot_next(s), comp);
        int p[3], ax;
        if (r < fz) {
            const int64_t half = (int64_t)(nx - 2) * (ny - 2);
            ax = 2;
            p[2] = r < half ? 0 : nz - 1;
            if (r >= half)
                r -= half;
            const uint32_t q = face_div(r, half, nx - 2);
            p[0] = 1 + (int)(r - (int64_t)q * (nx - 2));
            p[1] = 1 + (int)q;
        } else if (r < fz + fy) {
            r -= fz;
            const int64_t half = (int64_t)(nx - 2) * (nz - 2);
            ax = 1;
            p[1] = r < half ? 0 : ny - 1;
            if (r >= half)
                r -= half;
            const uint32_t q = face_div(r, half, nx - 2);
            p[0] = 1 + (int)(r - (int64_t)q * (nx - 2));
            p[2] = 1 + (int)q;
        } else {
            r -= fz + fy;
            const int64_t half = (int64_t)(ny - 2) * (nz - 2);
            ax = 0;
            p[0] = r < half ? 0 : nx - 1;
            if (r >= half)
                r -= half;
            const uint32_t q = face_div(r, half, ny - 2);
            p[1] = 1 + (int)(r - (int64_t)q * (ny - 2));
            p[2] = 1 + (int)q;
        }
        // strides of the normal axis by selects (no array indexed at run time)
        const int64_t sx = 1, sy = nx, sz = (int64_t)nx * ny;
        const int64_t sn = ax == 0 ? sx : (ax == 1 ? sy : sz);
        const int64_t s1 = ax == 0 ? sy : (ax == 1 ? sz : sx), s2 = ax == 0 ? sz : (ax == 1 ? sx : sy);
        const int pa = ax == 0 ? p[0] : (ax == 1 ? p[1] : p[2]);
        const int side = pa == 0 ? -1 : 1;
        const int64_t c = ((int64_t)p[2] * ny + p[1]) * nx + p[0];
        const int64_t q = c - side * sn;  // first node inside
        pp[c] = mur_face(R, ax, pm, p0, (double)pp[q], c, q, s1, s2);
    }
};


// ---------------------------------------------------------------------------
// K3: E and B at vertices
// ---------------------------------------------------------------------------

// The n+1 value of the boundary node beside interior node c0, one step of
// `side` along axis AX, from its face update (not from memory).
template <typename T, int AX>
__device__ inline double face_beside(const RunDev &R, int64_t s, int comp, int side, int64_t c0)
{
    const int64_t st[3] = {1, R.nx, (int64_t)R.nx * R.ny};
    return (double)mur_face(R, AX, pot_ptr<T>(R, slot_prev(s), comp), pot_ptr<T>(R, slot_cur(s), comp),
                            (double)pot_ptr<T>(R, slot_next(s), comp)[c0], c0 + side * st[AX], c0, st[(AX + 1) % 3],
                            st[(AX + 2) % 3]);
}

// E and B at interior node (i, j, k) from the levels n and n+1 of step s.
// FACES: the boundary's n+1 values are not there yet (the boundary update
// runs in the same launch), so a node beside the boundary computes the face
// values it needs.
template <typename T, bool FACES>
__device__ inline void vertex_eb(const RunDev &R, int64_t s, int i, int j, int k, double E[3], double B[3])
{
    const T *An[3], *Ap[3];
    for (int c = 0; c < 3; ++c) {
        An[c] = pot_ptr<T>(R, slot_cur(s), c);
        Ap[c] = pot_ptr<T>(R, slot_next(s), c);
    }
    const int64_t c0 = nid(R, i, j, k);
    const int64_t sx = 1, sy = R.nx, sz = (int64_t)R.nx * R.ny;
    const double i2x = 0.5 / R.dx, i2y = 0.5 / R.dy, i2z = 0.5 / R.dz;
    auto dif = [&](const T *a, int64_t st) { return (double)a[c0 + st] - (double)a[c0 - st]; };
    // differences of level n+1: A_z by y, A_y by z, A_x by z, A_z by x, A_y by x, A_x by y
    double zy = dif(Ap[2], sy), yz = dif(Ap[1], sz), xz = dif(Ap[0], sz), zx = dif(Ap[2], sx), yx = dif(Ap[1], sx),
           xy = dif(Ap[0], sy);
    if constexpr (FACES) {
        // the difference d of component c along an axis beside its face
        auto fix = [&](double &d, int side, double face, const T *a, int64_t st) {
            d = side < 0 ? (double)a[c0 + st] - face : face - (double)a[c0 - st];
        };
        if (j == 1 || j == R.ny - 2) {
            const int side = j == 1 ? -1 : 1;
            const double f2 = face_beside<T, 1>(R, s, 2, side, c0), f0 = face_beside<T, 1>(R, s, 0, side, c0);
            fix(zy, side, f2, Ap[2], sy);
            fix(xy, side, f0, Ap[0], sy);
        }
        if (k == 1 || k == R.nz - 2) {
            const int side = k == 1 ? -1 : 1;
            const double f1 = face_beside<T, 2>(R, s, 1, side, c0), f0 = face_beside<T, 2>(R, s, 0, side, c0);
            fix(yz, side, f1, Ap[1], sz);
            fix(xz, side, f0, Ap[0], sz);
        }
        if (!R.xface_fused && (i == 1 || i == R.nx - 2)) {
            const int side = i == 1 ? -1 : 1;
            const double f2 = face_beside<T, 0>(R, s, 2, side, c0), f1 = face_beside<T, 0>(R, s, 1, side, c0);
            fix(zx, side, f2, Ap[2], sx);
            fix(yx, side, f1, Ap[1], sx);
        }
    }
    // curl of A at n and at n+1, averaged
    B[0] = 0.5 * ((dif(An[2], sy) + zy) * i2y - (dif(An[1], sz) + yz) * i2z);
    B[1] = 0.5 * ((dif(An[0], sz) + xz) * i2z - (dif(An[2], sx) + zx) * i2x);
    B[2] = 0.5 * ((dif(An[1], sx) + yx) * i2x - (dif(An[0], sy) + xy) * i2y);
    double g[3] = {0.0, 0.0, 0.0};
    if (R.space_charge) {
        const T *ph = pot_ptr<T>(R, slot_cur(s), 3);
        g[0] = dif(ph, sx) * i2x;
        g[1] = dif(ph, sy) * i2y;
        g[2] = dif(ph, sz) * i2z;
    }
    for (int c = 0; c < 3; ++c)
        E[c] = -((double)Ap[c][c0] - (double)An[c][c0]) / R.dt - g[c];
}

// E, B over the active-particle box of the last push, where a particle
// gathers (FACES: see vertex_eb).
template <typename T, bool FACES>
struct VertexFields {
    static constexpr int kThreads = 256;
    static __device__ void run(const RunDev &R, Blk blk)
    {
        const int64_t s = R.ctl->step;
        int lo[3], hi[3];
        const int n[3] = {R.nx, R.ny, R.nz};
        for (int a = 0; a < 3; ++a) {
            lo[a] = max(1, R.ctl->cell_lo[a]);
            hi[a] = min(n[a] - 2, R.ctl->cell_hi[a] + 1);
            if (hi[a] < lo[a])
                return;
        }
        constexpr int V = 16 / sizeof(T);
        const BoxNodes box(lo[0], lo[1], lo[2], hi[0] - lo[0] + 1, hi[1] - lo[1] + 1, hi[2] - lo[2] + 1);
        for (int64_t t = (int64_t)blk.id * blockDim.x + threadIdx.x; t < box.tot; t += (int64_t)blk.n * blockDim.x) {
            int i, j, k;
            box.node(t, i, j, k);
            if (!node_marked(R, s, 0, i, j, k))
                continue;  // no particle of this step gathers at this node
            double E[3], B[3];
            vertex_eb<T, FACES>(R, s, i, j, k, E, B);
            Vec<T, V> w[8 / V];
            const T all[8] = {(T)E[0], (T)E[1], (T)E[2], (T)B[0], (T)B[1], (T)B[2], (T)0, (T)0};
            for (int q = 0; q < 8; ++q)
                w[q / V].v[q % V] = all[q];
            T *dst = eb_node<T>(R, nid(R, i, j, k));
            for (int q = 0; q < 8 / V; ++q)
                vstore<T, V>(dst + q * V, w[q]);
        }
    }
};

// Radiated power through node plane k_plane of the fields at t_{s+1/2}
// (lab-frame Poynting flux).  kPowerBlocks blocks write partial sums over
// a fixed node partition; one block adds them in fixed order, so the
// result does not depend on scheduling.  (A single launch whose last block
// adds the partial sums needs a device-scope release fence in every block,
// which writes back the XCD's L2: in a grouped launch of 32 runs that made
// the stage six times slower.)
template <typename T, bool FACES>
struct PlanePower {
    static constexpr int kThreads = 256;
    static __device__ void run(const RunDev &R, Blk blk, int step_bias, int kp_arg)
    {
        __shared__ double red[256];
        const int kp = kp_arg < 0 ? R.k_plane : kp_arg;  // < 0: the run's diagnostic plane
        const int64_t s = R.ctl->step + step_bias;
        const double g0 = R.gamma0, b0 = R.beta0;
        double acc = 0.0;
        const int wx = R.nx - 2, wy = R.ny - 2;
        for (int t = blk.id * 256 + threadIdx.x; t < wx * wy; t += kPowerBlocks * 256) {
            const int i = 1 + t % wx, j = 1 + t / wx;
            double E[3], B[3];
            vertex_eb<T, FACES>(R, s, i, j, kp, E, B);
            const double Exl = g0 * (E[0] + b0 * kC * B[1]);
            const double Eyl = g0 * (E[1] - b0 * kC * B[0]);
            const double Bxl = g0 * (B[0] - b0 * E[1] / kC);
            const double Byl = g0 * (B[1] + b0 * E[0] / kC);
            acc += Exl * Byl - Eyl * Bxl;
        }
        red[threadIdx.x] = acc;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w)
                red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0)
            R.ppart[blk.id] = red[0];
    }
};

struct PlanePowerFinal {
    static constexpr int kThreads = 64;
    static __device__ void run(const RunDev &R, Blk blk, int step_bias, double *out)
    {
        plane_power_final(R, R.ctl->step + step_bias, out, 0);
    }
};

// Workgroups of the vertex fields: an eighth of what one node per thread
// needs, 1024 at most.  The particle box is usually a small part of the grid
// (the grid holds the radiation around the bunch); workgroups past it find no
// node to do, but go through dispatch and hold the slots that the working ones
// and the boundary's wait for.  The grid-stride loop covers a box as large as
// the grid.  Single runs, the launch that holds them (StepFields), with up to
// 8192 / 2048 / 1024 workgroups: 128 x 128 x 1024 nodes FP32 89 / 79 / 80 us,
// FP64 133 / 123 / 122, 64 x 64 x 2800 FP64 143 / 133 / 131, 64 x 64 x 384
// 25 / 21 / 19.
__host__ __device__ inline int64_t vertex_blocks_of(const RunDev &R)
{
    const int64_t inner = (int64_t)(R.nx - 2) * (R.ny - 2) * (R.nz - 2);
    const int64_t b = (inner + 255) / 256 / 8;
    return b < 1 ? 1 : (b > 1024 ? 1024 : b);
}

// A run of its own: one node per thread up to two workgroups a CU, which are
// free slots on a device that runs nothing else.  With particles over the
// whole grid an eighth left CUs idle and each thread eight nodes in sequence:
// 32 x 32 x 64 FP32 50.2 -> 43.0 us a step (48.9 with one node per thread
// throughout, before StepFields), FP64 63.0 -> 54.5, 24 x 24 x 400 FP32 60.7 ->
// 49.5, 48 x 48 x 96 FP64 62.3 -> 54.4, 64 x 64 x 128 FP32 123 -> 119; with the
// bunch in a sixteenth of the grid across the same (34.7 and 39.2 us both).  One
// node per thread up to 1024 workgroups: 64 x 64 x 128 FP64 156 against 153.
static int64_t vertex_blocks_own(const RunDev &R)
{
    const int64_t inner = (int64_t)(R.nx - 2) * (R.ny - 2) * (R.nz - 2);
    const int64_t full = (inner + 255) / 256;
    const int64_t least = full < 512 ? full : 512, eighth = vertex_blocks_of(R);
    return eighth > least ? eighth : least;
}

// ---------------------------------------------------------------------------
// Spectral radiated power: running Fourier transforms over the boosted time
// t_{s+1/2} of the lab-frame E'_x E'_y B'_x B'_y at every interior node of
// the power plane, at omega_f = nu_f omega_r.  One thread per plane node
// owns its accumulators (no atomics); the fields are those of the plane
// power, from the potentials of step s.
// ---------------------------------------------------------------------------

__host__ __device__ inline double spec_nu(const RunDev &R, int f)
{
    return R.nfreq == 1 ? R.nu_min : R.nu_min + (R.nu_max - R.nu_min) * f / (double)(R.nfreq - 1);
}

template <typename T, bool FACES>
struct PlaneSpectrum {
    static constexpr int kThreads = 256;
    static __device__ void run(const RunDev &R, Blk blk)
    {
        const int64_t s = R.ctl->step;
        const int wx = R.nx - 2, wy = R.ny - 2;
        const int t = (int)(blk.id * kThreads + threadIdx.x);
        if (t >= wx * wy)
            return;
        const int i = 1 + t % wx, j = 1 + t / wx;
        double E[3], B[3];
        vertex_eb<T, FACES>(R, s, i, j, R.k_plane, E, B);
        const double g0 = R.gamma0, b0 = R.beta0;
        double F[4];
        F[0] = g0 * (E[0] + b0 * kC * B[1]);
        F[1] = g0 * (E[1] - b0 * kC * B[0]);
        F[2] = g0 * (B[0] - b0 * E[1] / kC);
        F[3] = g0 * (B[1] + b0 * E[0] / kC);
        const double tt = ((double)s + 0.5) * R.dt;
        const int64_t plane = (int64_t)R.nx * R.ny, pidx = (int64_t)j * R.nx + i;
        for (int f = 0; f < R.nfreq; ++f) {
            const double om = spec_nu(R, f) * R.omega_r;
            const double c = cos(om * tt) * R.dt, sn = -sin(om * tt) * R.dt;
            double *acc = R.spec + (int64_t)f * 8 * plane + pidx;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[(2 * q) * plane] += F[q] * c;
                acc[(2 * q + 1) * plane] += F[q] * sn;
            }
        }
    }
};

__host__ __device__ inline int64_t spectrum_blocks_of(const RunDev &R)
{
    return R.nfreq > 0 ? ((int64_t)(R.nx - 2) * (R.ny - 2) + 255) / 256 : 0;
}

// A single run's stages between the sweep and the push in one launch: the
// plane power's partial sums, the plane spectrum, the boundary faces with the
// clearing of the next source set, and the vertex fields.  The power, the
// spectrum and the vertex fields read the potentials of step s only, and
// where they need the boundary's n+1 values they compute them (vertex_eb),
// so nothing here waits for anything else here.  With the faces in a launch
// before and the spectrum in one after: 64 x 64 x 256 FP64 with the spectrum
// 92 -> 82 us a step, 32 x 32 x 64 FP64 39.9 -> 38.0, 64 x 64 x 2800 FP64 512
// -> 494, 128 x 128 x 1024 FP32 430 -> 422 (entrance phase).
// The short dependent chains come first, so that they do not form the
// launch's tail, the boundary's plain streams last (before the vertex fields:
// 80 -> 93 us at 128 x 128 x 1024 FP32).  Grouped steps launch the boundary
// by itself (VertexPower): the face values cost the vertex fields registers,
// and a step of 16 runs took 537 us with this body and 515 without.
template <typename T>
struct StepFields {
    static constexpr int kThreads = 256;
    static __host__ __device__ int64_t power_blocks(const RunDev &R) { return R.record_power ? kPowerBlocks : 0; }
    static __device__ void run(const RunDev &R, Blk blk)
    {
        const int64_t np = power_blocks(R), ns = spectrum_blocks_of(R), nm = mur_blocks_of(R);
        if (blk.id == 0 && threadIdx.x == 0)
            R.ctl->next_step = R.ctl->step + 1;
        if (blk.id < np)
            PlanePower<T, true>::run(R, Blk{blk.id, kPowerBlocks}, 0, -1);
        else if (blk.id < np + ns)
            PlaneSpectrum<T, true>::run(R, Blk{blk.id - np, ns});
        else if (blk.id < blk.n - nm)
            VertexFields<T, true>::run(R, Blk{blk.id - np - ns, blk.n - np - ns - nm});
        else
            Mur<T>::run(R, Blk{blk.id - (blk.n - nm), nm});
    }
};

// dW/domega of frequency f = blockIdx.x: (1/pi) (dx dy / mu0) sum over the
// plane's interior nodes of Re(Ex' By'* - Ey' Bx'*), fixed-order tree sum
__global__ __launch_bounds__(256) void k_spec_reduce(RunDev R, double *out)
{
    __shared__ double red[256];
    const int f = blockIdx.x;
    const int wx = R.nx - 2, wy = R.ny - 2;
    const int64_t plane = (int64_t)R.nx * R.ny;
    const double *acc = R.spec + (int64_t)f * 8 * plane;
    double sum = 0.0;
    for (int t = threadIdx.x; t < wx * wy; t += 256) {
        const int64_t p = (int64_t)(1 + t / wx) * R.nx + 1 + t % wx;
        sum += (acc[0 * plane + p] * acc[6 * plane + p] + acc[1 * plane + p] * acc[7 * plane + p]) -
               (acc[2 * plane + p] * acc[4 * plane + p] + acc[3 * plane + p] * acc[5 * plane + p]);
    }
    red[threadIdx.x] = sum;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double mu0 = 1.0 / (kEps0 * kC * kC);
        out[f] = red[0] * R.dx * R.dy / (mu0 * kPi);
    }
}

// ---------------------------------------------------------------------------
// TF/SF seed injection on the planes k = 1 (scattered-field boundary) and
// k = 2 (total-field boundary): after the update of A_x and A_y, each node
// gets back the incident-wave part of the terms through which it used the
// other region's values, so that the total-field region holds +f.
// Incident wave (boosted, along +z): A = A0 p s(t - (z - z_2)/c), the lab
// signal Doppler-scaled by gamma0 (1 + beta0); Gaussian seeds add the
// paraxial amplitude, curvature and Gouy phase.
// ---------------------------------------------------------------------------

// The incident wave on one plane: everything but the radius is uniform on
// it.  F(r2) = a (without the polarisation) exp(-r2 / w2) cos(ph + curv r2).
struct SeedPlane {
    double a, w2, ph, curv;
};

__device__ inline SeedPlane seed_plane(const RunDev &R, int k, double t)
{
    const double z = R.z0 + k * R.dz, z2 = R.z0 + 2.0 * R.dz;
    const double D = R.gamma0 * (1.0 + R.beta0);
    const double lam = R.seed_lambda * D;
    const double f = kC / lam, tp = R.seed_ctau / kC * D, t0 = R.seed_ct0 / kC * D;
    const double d = t - (z - z2) / kC - t0;
    const double ln2 = 0.69314718055994530942;
    SeedPlane P{R.seed_a0 * kMe * kC / kQe, 1.0, 2.0 * kPi * f * d + R.seed_cep, 0.0};
    // the signal's envelope (the carrier is the cosine of F)
    const double gauss = exp(-2.0 * ln2 * d * d / (tp * tp));
    if (R.seed_signal == 0)
        P.a *= -4.0 * ln2 * (d / tp) * gauss;
    else if (R.seed_signal == 1 || (R.seed_signal == 3 && d <= 0.0))
        P.a *= gauss;
    else if (R.seed_signal == 2)
        P.a *= 1.0 / cosh(d / tp);
    if (R.seed_type == 1) {
        const double zR = kPi * R.seed_w0 * R.seed_w0 / lam;
        const double l = z - R.seed_zf;
        const double w = R.seed_w0 * sqrt(1.0 + (l / zR) * (l / zR));
        P.a *= R.seed_w0 / w;
        P.w2 = w * w;
        P.curv = -0.5 * (2.0 * kPi / lam) * l / (l * l + zR * zR);
        P.ph += atan(l / zR);
    }
    return P;
}

// Bound by latency (two planes of nodes; FP64 exp and cos).  A workgroup
// takes a 32 x 8 tile of both planes and both components: the wave on the
// tile and its one-node halo is evaluated once into LDS (the components
// differ by the polarisation only), where each node and component evaluated
// ten neighbours itself: 64 x 64 nodes 22.9 us a launch, now 10.2.
// With the x faces fused into the sweep (xface_fused) the face nodes beside
// a corrected node are computed again from its new value, so a seeded run
// takes the vector sweep: the scalar one and the boundary kernel's x faces
// cost 30 + 15 us more at 64 x 64 x 384 nodes.
template <typename T>
struct SeedInject {
    static constexpr int kThreads = 256;
    static constexpr int TX = 32, TY = 8;
    static __device__ void run(const RunDev &R, Blk blk)
    {
        __shared__ SeedPlane P[2];
        __shared__ double F[2][TY + 2][TX + 2];
        const int64_t s = R.ctl->step;
        const int wx = R.nx - 2, wy = R.ny - 2;
        const int ntx = (wx + TX - 1) / TX;
        const int i0 = (int)(blk.id % ntx) * TX, j0 = (int)(blk.id / ntx) * TY;  // node left of and below the tile
        if (threadIdx.x < 2)
            P[threadIdx.x] = seed_plane(R, 1 + (int)threadIdx.x, (double)s * R.dt);  // time level n of the update
        __syncthreads();
        for (int e = threadIdx.x; e < 2 * (TY + 2) * (TX + 2); e += kThreads) {
            const int pl = e / ((TY + 2) * (TX + 2)), r = e - pl * ((TY + 2) * (TX + 2));
            const int ej = r / (TX + 2), ei = r - ej * (TX + 2);
            const double x = R.x0 + (i0 + ei) * R.dx, y = R.y0 + (j0 + ej) * R.dy;
            const double r2 = x * x + y * y;
            const SeedPlane p = P[pl];
            double v = p.a * cos(p.ph + p.curv * r2);
            if (R.seed_type == 1)
                v *= exp(-r2 / p.w2);
            F[pl][ej][ei] = v;
        }
        __syncthreads();
        const int li = 1 + (int)(threadIdx.x % TX), lj = 1 + (int)(threadIdx.x / TX);
        const int i = i0 + li, j = j0 + lj;
        if (i > wx || j > wy)
            return;
        // plane 1 loses the wave that it read from plane 2, plane 2 gets the one that plane 1 lacks
        double corr[2];
        for (int pl = 0; pl < 2; ++pl) {
            const double(*f)[TX + 2] = F[1 - pl];
            const double c = R.A * (R.a2 * f[lj][li + 1] + R.a2 * f[lj][li - 1] + R.a4 * f[lj + 1][li] +
                                    R.a4 * f[lj - 1][li]) + R.a6 * f[lj][li];
            corr[pl] = pl == 0 ? -c : c;
        }
        double pol[2];
        sincos(R.seed_pol, &pol[1], &pol[0]);
        const int64_t sy = R.nx, sz = (int64_t)R.nx * R.ny;
        for (int comp = 0; comp < 2; ++comp) {
            T *pn = pot_ptr<T>(R, slot_next(s), comp);
            const T *p0 = pot_ptr<T>(R, slot_cur(s), comp), *pm = pot_ptr<T>(R, slot_prev(s), comp);
            for (int pl = 0; pl < 2; ++pl) {
                const int64_t n = nid(R, i, j, 1 + pl);
                const T v = (T)((double)pn[n] + pol[comp] * corr[pl]);
                pn[n] = v;
                for (int side = -1; side <= 1; side += 2)
                    if (R.xface_fused && i == (side < 0 ? 1 : wx))
                        pn[n + side] = mur_face(R, 0, pm, p0, (double)v, n + side, n, sy, sz);
            }
        }
    }
};

__host__ __device__ inline int64_t seed_blocks_of(const RunDev &R)
{
    return (int64_t)((R.nx - 2 + 31) / 32) * ((R.ny - 2 + 7) / 8);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------

// Potentials that a sweep advances: phi only with space charge.  It is the
// slowest index of the tiles, of which each XCD takes a contiguous eighth, so
// workgroups for a phi that is not advanced would leave two of the eight idle:
// 72 x 56 x 136 FP64 without space charge 44.7 -> 42.3 us a step, 64 x 64 x 256
// FP64 71.6 -> 67.9, 128 x 128 x 1024 FP32 302 -> 295, 64 x 64 x 2800 FP64 454 ->
// 452 (bound by its bytes on any number of XCDs).
static int sweep_components(int space_charge) { return space_charge ? 4 : 3; }

template <typename T, int TX, int TY, int TZ>
static hipError_t launch_sweep_t(const RunDev &R, hipStream_t st)
{
    const int64_t ntx = (R.nx + TX - 1) / TX, nty = (R.ny + TY - 1) / TY;
    const int64_t nch = (R.nz - 2 + TZ - 1) / TZ;
    const int64_t nb = ntx * nty * nch * sweep_components(R.space_charge);
    hipLaunchKernelGGL((k_run<Sweep<T, TX, TY, TZ>>), dim3((unsigned)nb), dim3(TX * TY), 0, st, R);
    return hipGetLastError();
}

template <typename T, int V, int TXV, int TY, int TZ>
static hipError_t launch_sweep_vec_t(const RunDev &R, int tail, hipStream_t st)
{
    constexpr int TW = TXV * V;
    const int64_t ntx = (R.nx + TW - 1) / TW, nty = (R.ny + TY - 1) / TY;
    const int64_t nch = (R.nz - 2 + TZ - 1) / TZ;
    const dim3 grid((unsigned)(ntx * nty * nch * sweep_components(R.space_charge) + tail)), block(TXV * TY);
    if constexpr (sizeof(T) == 4) {
        if (R.compensated) {
            hipLaunchKernelGGL((k_run<SweepWithTail<SweepVec<T, V, TXV, TY, TZ, true>>, int>), grid, block, 0, st, R,
                               tail);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_run<SweepWithTail<SweepVec<T, V, TXV, TY, TZ, false>>, int>), grid, block, 0, st, R, tail);
    return hipGetLastError();
}

// Tiles of the sweep: x nodes, y rows (FP32; the vector tiles' rows halve at
// FP64), z planes.  0..7 scalar (one node per thread), 8..17 vector (16
// bytes per thread).  Workgroups of 256 threads, 5 and 12 of 512: other
// tiles of 512 threads were slower on grids that leave CUs idle and no
// faster on large ones (in the step of the 128 x 128 x 1024 run: 64 x 32 x
// 16 nodes in 512 threads 166 us at FP32 and 309 at FP64, 64 x 16 x 16 in
// 256 162 and 302; tiles over 32 or 64 planes 169 and more).
static const int kSweepTile[18][3] = {{64, 4, 16}, {64, 4, 4},  {32, 8, 4},  {64, 4, 8},   {32, 8, 8},   {64, 8, 32},
                                      {32, 8, 16}, {16, 16, 4}, {16, 64, 4}, {32, 32, 4},  {32, 32, 8},  {32, 32, 16},
                                      {128, 16, 8}, {64, 16, 4}, {64, 16, 8}, {64, 16, 16}, {128, 8, 4}, {128, 8, 16}};

int sweep_shape_count() { return 18; }

// Vector tiles need rows that start on 16 bytes.
static bool sweep_aligned(int nx, int precision) { return nx % (precision == 32 ? 4 : 2) == 0; }

// tiles of one component
static int64_t sweep_tiles(int nx, int ny, int nz, int precision, int shape)
{
    const int *d = kSweepTile[shape];
    const int ty = shape >= 8 && precision == 64 ? d[1] / 2 : d[1];
    return (int64_t)((nx + d[0] - 1) / d[0]) * ((ny + ty - 1) / ty) * ((nz - 2 + d[2] - 1) / d[2]);
}

// Default tile of a grid: the least estimated time, in units of one plane of
// a workgroup (about 0.4 us), from what bounds a sweep:
//  * the planes that the workgroups run one after the other: rounds of
//    resident workgroups (at least one) times the planes of a tile and its
//    prologue.  Few planes fill the device on a small grid;
//  * the bytes of a node: three streams, and psi^n again for each tile's
//    two extra planes, its halo rows and the partly used vectors at its
//    row ends.  Many planes and wide tiles read less on a large grid.
// The constants were fitted on 70 aligned and 40 unaligned grids (12..129 x
// 12..128 x 40..2800, both precisions, every tile timed): the choice is
// within 3 % of the best tile in the mean and 25 % at worst; the earlier rule
// (two tiles by the node count, a third for short rows) was 35 % off in the
// mean.  Sweep alone, before and after: 64 x 64 x 256 FP64 37.4 -> 21.5 us,
// 96 x 80 x 192 FP32 31.3 -> 21.4, 24 x 24 x 400 FP32 19.5 -> 8.8, 45 x 51 x
// 97 FP32 19.9 -> 9.0; in the step of the 128 x 128 x 1024 run FP32 166 -> 162,
// FP64 309 -> 302.  Without space charge there are three components to count:
// with four, 4 of 60 grids took another tile and were 15 % from the best one in
// the mean, with three 2 % (112 x 54 x 167 FP32 14.1 -> 11.6 us, 57 x 25 x 772
// FP64 23.6 -> 17.5).
int sweep_default_shape(int nx, int ny, int nz, int precision, int space_charge)
{
    const bool vec = sweep_aligned(nx, precision);
    const double slots = vec ? 576 : 1500, prologue = vec ? 1.5 : 0.5, row_end = vec ? 24 : 8;
    const int comps = sweep_components(space_charge);
    const double mb = 1e-6 * comps * nx * ny * nz * (precision / 8);
    int best = -1;
    double best_cost = 0;
    for (int s = vec ? 8 : 0; s < (vec ? 18 : 8); ++s) {
        const int *d = kSweepTile[s];
        const double ty = vec && precision == 64 ? d[1] / 2 : d[1], tz = d[2];
        const double n = (double)comps * sweep_tiles(nx, ny, nz, precision, s) * (s == 5 || s == 12 ? 2 : 1);
        const double cost = std::max(1.0, n / slots) * (tz + prologue) +
                            mb * (3 + 2 / tz + 5 / ty * (1 + 2 / tz) + row_end / d[0]) / 13;
        if (best < 0 || cost < best_cost) {
            best = s;
            best_cost = cost;
        }
    }
    return best;
}

// The tile that runs for a chosen one: a vector tile on unaligned rows is
// replaced by the grid's default (scalar) tile.
int sweep_effective_shape(const RunDev &R, int shape)
{
    if (shape >= 8 && !sweep_aligned(R.nx, R.precision))
        return sweep_default_shape(R.nx, R.ny, R.nz, R.precision, R.space_charge);
    return shape;
}

int sweep_fuses_xfaces(const RunDev &R, int shape) { return shape >= 8 && sweep_aligned(R.nx, R.precision) ? 1 : 0; }

template <typename T>
static hipError_t launch_sweep_shape(const RunDev &R, int shape, int tail, hipStream_t st)
{
    constexpr int V = 16 / sizeof(T);
    switch (sweep_effective_shape(R, shape)) {
    case 8: return launch_sweep_vec_t<T, V, 16 / V, 256 * V / 16, 4>(R, tail, st);
    case 9: return launch_sweep_vec_t<T, V, 32 / V, 256 * V / 32, 4>(R, tail, st);
    case 10: return launch_sweep_vec_t<T, V, 32 / V, 256 * V / 32, 8>(R, tail, st);
    case 11: return launch_sweep_vec_t<T, V, 32 / V, 256 * V / 32, 16>(R, tail, st);
    case 12: return launch_sweep_vec_t<T, V, 128 / V, 512 * V / 128, 8>(R, tail, st);
    case 13: return launch_sweep_vec_t<T, V, 64 / V, 256 * V / 64, 4>(R, tail, st);
    case 14: return launch_sweep_vec_t<T, V, 64 / V, 256 * V / 64, 8>(R, tail, st);
    case 15: return launch_sweep_vec_t<T, V, 64 / V, 256 * V / 64, 16>(R, tail, st);
    case 16: return launch_sweep_vec_t<T, V, 128 / V, 256 * V / 128, 4>(R, tail, st);
    case 17: return launch_sweep_vec_t<T, V, 128 / V, 256 * V / 128, 16>(R, tail, st);
    case 0: return launch_sweep_t<T, 64, 4, 16>(R, st);
    case 1: return launch_sweep_t<T, 64, 4, 4>(R, st);
    case 2: return launch_sweep_t<T, 32, 8, 4>(R, st);
    case 3: return launch_sweep_t<T, 64, 4, 8>(R, st);
    case 4: return launch_sweep_t<T, 32, 8, 8>(R, st);
    case 5: return launch_sweep_t<T, 64, 8, 32>(R, st);
    case 6: return launch_sweep_t<T, 32, 8, 16>(R, st);
    case 7: return launch_sweep_t<T, 16, 16, 4>(R, st);
    default: return hipErrorInvalidValue;
    }
}

// tail: the launch also ends the step before (vector tiles only)
hipError_t launch_sweep(const RunDev &R, int shape, hipStream_t st, int tail)
{
    if (tail && !sweep_fuses_xfaces(R, shape))
        return hipErrorInvalidValue;
    return R.precision == 32 ? launch_sweep_shape<float>(R, shape, tail, st)
                             : launch_sweep_shape<double>(R, shape, tail, st);
}

int64_t mur_blocks(const RunDev &R) { return mur_blocks_of(R); }

// Mur edge and corner workgroups (per component)
int64_t mur_edge_blocks(const RunDev &R) { return mur_edge_blocks_of(R); }

hipError_t launch_mur(const RunDev &R, hipStream_t st)
{
    const unsigned blocks = (unsigned)mur_blocks(R), eblocks = (unsigned)mur_edge_blocks(R);
    if (R.precision == 32) {
        hipLaunchKernelGGL((k_run<Mur<float>>), dim3(blocks), dim3(256), 0, st, R);
        hipLaunchKernelGGL((k_run<MurEdge<float>>), dim3(eblocks), dim3(256), 0, st, R);
    } else {
        hipLaunchKernelGGL((k_run<Mur<double>>), dim3(blocks), dim3(256), 0, st, R);
        hipLaunchKernelGGL((k_run<MurEdge<double>>), dim3(eblocks), dim3(256), 0, st, R);
    }
    return hipGetLastError();
}

hipError_t launch_step_fields(const RunDev &R, hipStream_t st)
{
    const unsigned blocks = (unsigned)(StepFields<float>::power_blocks(R) + spectrum_blocks_of(R) + mur_blocks_of(R) +
                                       vertex_blocks_own(R));
    if (R.precision == 32)
        hipLaunchKernelGGL((k_run<StepFields<float>>), dim3(blocks), dim3(256), 0, st, R);
    else
        hipLaunchKernelGGL((k_run<StepFields<double>>), dim3(blocks), dim3(256), 0, st, R);
    return hipGetLastError();
}

hipError_t launch_spec_reduce(const RunDev &R, double *out, hipStream_t st)
{
    if (R.nfreq <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_spec_reduce, dim3((unsigned)R.nfreq), dim3(256), 0, st, R, out);
    return hipGetLastError();
}

hipError_t launch_seed_inject(const RunDev &R, hipStream_t st)
{
    if (!R.seed_on)
        return hipSuccess;
    const unsigned nb = (unsigned)seed_blocks_of(R);
    if (R.precision == 32)
        hipLaunchKernelGGL((k_run<SeedInject<float>>), dim3(nb), dim3(256), 0, st, R);
    else
        hipLaunchKernelGGL((k_run<SeedInject<double>>), dim3(nb), dim3(256), 0, st, R);
    return hipGetLastError();
}

hipError_t launch_plane_power(const RunDev &R, int step_bias, int kp, double *out, hipStream_t st)
{
    if (R.precision == 32)
        hipLaunchKernelGGL((k_run<PlanePower<float, false>, int, int>), dim3(kPowerBlocks), dim3(256), 0, st, R, step_bias, kp);
    else
        hipLaunchKernelGGL((k_run<PlanePower<double, false>, int, int>), dim3(kPowerBlocks), dim3(256), 0, st, R, step_bias, kp);
    hipLaunchKernelGGL((k_run<PlanePowerFinal, int, double *>), dim3(1), dim3(64), 0, st, R, step_bias, out);
    return hipGetLastError();
}

}  // namespace mithra

// ---------------------------------------------------------------------------
// grouped launches (several runs per launch; see k_group)
// ---------------------------------------------------------------------------
namespace mithra {

int64_t sweep_blocks(const RunDev &R, int shape)
{
    return sweep_tiles(R.nx, R.ny, R.nz, R.precision, sweep_effective_shape(R, shape)) * sweep_components(R.space_charge);
}

template <typename T, int TX, int TY, int TZ>
static void grp_sweep_t(const Group &g, int64_t total, hipStream_t st)
{
    hipLaunchKernelGGL((k_group<Sweep<T, TX, TY, TZ>>), dim3((unsigned)total), dim3(TX * TY), 0, st, g);
}

template <typename T, int V, int TXV, int TY, int TZ>
static void grp_sweep_vec_t(const Group &g, int64_t total, bool lo, hipStream_t st)
{
    if constexpr (sizeof(T) == 4) {
        if (lo) {
            hipLaunchKernelGGL((k_group<SweepVec<T, V, TXV, TY, TZ, true>>), dim3((unsigned)total), dim3(TXV * TY), 0,
                               st, g);
            return;
        }
    }
    hipLaunchKernelGGL((k_group<SweepVec<T, V, TXV, TY, TZ, false>>), dim3((unsigned)total), dim3(TXV * TY), 0, st, g);
}

template <typename T>
static hipError_t grp_sweep(const Group &g, int64_t total, int shape, bool lo, hipStream_t st)
{
    constexpr int V = 16 / sizeof(T);
    switch (shape) {
    case 8: grp_sweep_vec_t<T, V, 16 / V, 256 * V / 16, 4>(g, total, lo, st); break;
    case 9: grp_sweep_vec_t<T, V, 32 / V, 256 * V / 32, 4>(g, total, lo, st); break;
    case 10: grp_sweep_vec_t<T, V, 32 / V, 256 * V / 32, 8>(g, total, lo, st); break;
    case 11: grp_sweep_vec_t<T, V, 32 / V, 256 * V / 32, 16>(g, total, lo, st); break;
    case 12: grp_sweep_vec_t<T, V, 128 / V, 512 * V / 128, 8>(g, total, lo, st); break;
    case 13: grp_sweep_vec_t<T, V, 64 / V, 256 * V / 64, 4>(g, total, lo, st); break;
    case 14: grp_sweep_vec_t<T, V, 64 / V, 256 * V / 64, 8>(g, total, lo, st); break;
    case 15: grp_sweep_vec_t<T, V, 64 / V, 256 * V / 64, 16>(g, total, lo, st); break;
    case 16: grp_sweep_vec_t<T, V, 128 / V, 256 * V / 128, 4>(g, total, lo, st); break;
    case 17: grp_sweep_vec_t<T, V, 128 / V, 256 * V / 128, 16>(g, total, lo, st); break;
    case 0: grp_sweep_t<T, 64, 4, 16>(g, total, st); break;
    case 1: grp_sweep_t<T, 64, 4, 4>(g, total, st); break;
    case 2: grp_sweep_t<T, 32, 8, 4>(g, total, st); break;
    case 3: grp_sweep_t<T, 64, 4, 8>(g, total, st); break;
    case 4: grp_sweep_t<T, 32, 8, 8>(g, total, st); break;
    case 5: grp_sweep_t<T, 64, 8, 32>(g, total, st); break;
    case 6: grp_sweep_t<T, 32, 8, 16>(g, total, st); break;
    case 7: grp_sweep_t<T, 16, 16, 4>(g, total, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// all members share precision, compensation and the (effective) shape
hipError_t launch_sweep_group(const Group &g, int64_t total, int precision, int compensated, int shape,
                              hipStream_t st)
{
    if (total <= 0)
        return hipSuccess;
    return precision == 32 ? grp_sweep<float>(g, total, shape, compensated != 0, st)
                           : grp_sweep<double>(g, total, shape, false, st);
}



// ge: the same members with their edge and corner workgroup counts
hipError_t launch_mur_group(const Group &g, int64_t total, const Group &ge, int64_t total_e, int precision,
                            hipStream_t st)
{
    if (total <= 0)
        return hipSuccess;
    if (precision == 32) {
        hipLaunchKernelGGL((k_group<Mur<float>>), dim3((unsigned)total), dim3(256), 0, st, g);
        if (total_e > 0)
            hipLaunchKernelGGL((k_group<MurEdge<float>>), dim3((unsigned)total_e), dim3(256), 0, st, ge);
    } else {
        hipLaunchKernelGGL((k_group<Mur<double>>), dim3((unsigned)total), dim3(256), 0, st, g);
        if (total_e > 0)
            hipLaunchKernelGGL((k_group<MurEdge<double>>), dim3((unsigned)total_e), dim3(256), 0, st, ge);
    }
    return hipGetLastError();
}

// Vertex fields and, beside them, the power's partial sums of each member;
// the power's few workgroups go first.  A step of 16 mixed runs (32 to 96
// nodes across, up to 256 along) took 521 us with two launches, 515 with one.
template <typename T>
struct VertexPower {
    static constexpr int kThreads = 256;
    static __device__ void run(const RunDev &R, Blk blk)
    {
        const int64_t np = StepFields<T>::power_blocks(R);
        if (blk.id < np)
            PlanePower<T, false>::run(R, Blk{blk.id, kPowerBlocks}, 0, -1);
        else
            VertexFields<T, false>::run(R, Blk{blk.id - np, blk.n - np});
    }
};

int64_t vertex_power_blocks(const RunDev &R) { return StepFields<float>::power_blocks(R) + vertex_blocks_of(R); }

hipError_t launch_vertex_power_group(const Group &g, int64_t total, int precision, hipStream_t st)
{
    if (total <= 0)
        return hipSuccess;
    if (precision == 32)
        hipLaunchKernelGGL((k_group<VertexPower<float>>), dim3((unsigned)total), dim3(256), 0, st, g);
    else
        hipLaunchKernelGGL((k_group<VertexPower<double>>), dim3((unsigned)total), dim3(256), 0, st, g);
    return hipGetLastError();
}

// After the pushes of all members: each member's box reductions (one
// workgroup) and its Mur edges and corners, which only have to be done before
// the step ends.  Neither reads what the other writes.  Edges that ran after
// the faces, a launch for each precision in the chain before the push, and the
// power's sum and the counters in two launches: 525 us a step of 16 mixed
// runs; with this and EndStep 521.
struct BoxEdges {
    static constexpr int kThreads = 256;
    static __device__ void run(const RunDev &R, Blk blk)
    {
        if (blk.id == 0)
            BoxReduceStep::run(R, blk);
        else if (R.precision == 32)
            MurEdge<float>::run(R, Blk{blk.id - 1, blk.n - 1});
        else
            MurEdge<double>::run(R, Blk{blk.id - 1, blk.n - 1});
    }
};

hipError_t launch_box_edges_group(const Group &g, int64_t total, hipStream_t st)
{
    if (total <= 0)
        return hipSuccess;
    hipLaunchKernelGGL((k_group<BoxEdges>), dim3((unsigned)total), dim3(256), 0, st, g);
    return hipGetLastError();
}

// The end of a member's step: the power from the partial sums, if recorded,
// and the bookkeeping.  One workgroup a member.
struct EndStep {
    static constexpr int kThreads = 64;
    static __device__ void run(const RunDev &R, Blk) { end_step(R); }
};

hipError_t launch_end_step_group(const Group &g, int64_t total, hipStream_t st)
{
    if (total <= 0)
        return hipSuccess;
    hipLaunchKernelGGL((k_group<EndStep>), dim3((unsigned)total), dim3(EndStep::kThreads), 0, st, g);
    return hipGetLastError();
}

}  // namespace mithra
