// Boundary coefficients and the Slater step on the first octant of a grid.
//
// The grid is symmetric about the expansion centre (the box centre), and each
// solid harmonic H_q = r^l Y_lm and each unit-moment boundary solution U_q
// (K U_q = the boundary term of moment vector e_q) keeps or flips sign under
// the reflection of an axis.  A contraction of a field with them over the
// grid is therefore one over the first octant, with the field folded into
// its eight parity classes (24 additions per eight nodes), and only the
// harmonics of a class meet that class: 49 products per eight nodes at
// lmax 6 instead of 392.  Likewise sum_q a_q H_q at the eight images of an
// octant node are eight sums over a class each, then 24 additions; the Slater
// step forms them once for each of the four images in y and z (a wave each, the
// signs on the operand), so 196 products per eight nodes and field.
//
// Two contractions with rho_i feed the rest of a step:
//   Q_q,i  = dV sum_n H_q rho_i      (the multipole moments),
//   zt_q,i = sum_n U_q rho_i         (the adjoint boundary coefficients:
//            zt_q = (1/4 pi) <C E e_q, w> = (1/4 pi) <K U_q, w> = <U_q, rho>,
//            since K is symmetric and K w = 4 pi rho),
// and give v_i = w_i + sum_q Q_q,i U_q and A^T rho_i = w_i + dV sum_q zt_q,i H_q
// from the zero-boundary solution w_i.
#include <algorithm>
#include <array>
#include <map>
#include <mutex>

#include "buffer.h"
#include "kernels.h"
#include "lds.h"
#include "lsda.h"

namespace fsic {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ dbl4 mfma(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Harmonics q = l^2 + l + mq (mq >= 0: Re (x + iy)^m, mq < 0: Im (x + iy)^m,
// m = |mq|, times a polynomial in z and r^2 of z-parity l - m) by parity
// class: bit 0 odd in x, bit 1 odd in y, bit 2 odd in z.  A class is padded
// to whole k steps of four.
template <int L>
struct Classes {
    int count[8];     // harmonics of a class
    int ks[9];        // k steps of classes 0 .. c - 1
    int row[8][16];   // harmonics in order (padding repeats the first)
};

constexpr int parity_of(int l, int mq) {
    const int m = mq < 0 ? -mq : mq;
    const int px = mq >= 0 ? (m & 1) : ((m + 1) & 1), py = mq >= 0 ? 0 : 1, pz = (l + m) & 1;
    // Im (x + iy)^m: odd in y, and odd in x where m is even
    return px | (py << 1) | (pz << 2);
}

template <int L>
constexpr Classes<L> make_classes() {
    Classes<L> t{};
    for (int l = 0; l <= L; ++l)
        for (int mq = -l; mq <= l; ++mq) {
            const int c = parity_of(l, mq);
            t.row[c][t.count[c]++] = l * l + l + mq;
        }
    for (int c = 0; c < 8; ++c) {
        t.ks[c + 1] = t.ks[c] + (t.count[c] + 3) / 4;
        for (int i = t.count[c]; i < 16; ++i) t.row[c][i] = t.row[c][0];
    }
    return t;
}

template <int L>
constexpr Classes<L> kCls = make_classes<L>();

template <int L>
constexpr int kSteps = kCls<L>.ks[8];

// The moments contract H and U with the same folded density: a 16-row
// operand holds up to eight harmonics of a class from H (rows 0-7) and the
// same ones from U (rows 8-15); slot k is harmonics first[k] .. of class
// cls[k].
template <int L>
struct Slots {
    int n, cls[16], first[16];
};
template <int L>
constexpr Slots<L> make_slots() {
    Slots<L> t{};
    for (int c = 0; c < 8; ++c)
        for (int f = 0; f < kCls<L>.count[c]; f += 8) {
            t.cls[t.n] = c;
            t.first[t.n++] = f;
        }
    return t;
}
template <int L>
constexpr Slots<L> kSlots = make_slots<L>();

// sum over the 16 lanes of a row, in a fixed order; every lane gets it
template <int R>
__device__ __forceinline__ double row_rotate(double v) {
    union {
        double d;
        int i[2];
    } a, b;
    a.d = v;
    b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], 0x120 + R, 0xf, 0xf, true);
    b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], 0x120 + R, 0xf, 0xf, true);
    return b.d;
}
__device__ __forceinline__ double row_sum(double v) {
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v += row_rotate<2>(v);
    v += row_rotate<1>(v);
    return v;
}

// octant coordinates of linear octant index o
__device__ __forceinline__ void oct_coords(int o, int hx, int hy, int &i, int &j, int &k) {
    const int r = o / hx;
    i = o - r * hx;
    k = r / hy;
    j = r - k * hy;
}

}  // namespace

// ---------------------------------------------------------------------------
// Q and zt of every orbital of a group (channels on one grid, consecutive
// fields): D[harmonic][orbital] += H or U[harmonic][node] rho_class[node]
// [orbital].  A block takes 16 orbitals and, 32 octant nodes at a time, loads
// their eight images along the nodes (whole lines), folds rho into the
// classes and turns it into the operand layout through LDS, with the 2 nlm
// rows of H and U beside it; its waves split the k steps.  The next tile's
// loads are in flight during the products.  Bound by the read of phi (8 B per
// orbital node) and of H and U (98 B a node and 16 orbitals at lmax 6, mostly
// from L2 when a grid has more than 16 orbitals).  Loading operands straight
// from memory (lanes along the orbitals) took 128 us at 96^3 with 31
// orbitals: 64 separate requests per load.  Orders 7 and 8 hold more
// accumulator tiles than there are registers (124 and 340 B a lane spilled; a
// whole step of these orbitals 1.46 and 1.77 ms, 1.38 at order 6).
// ---------------------------------------------------------------------------
constexpr int kOmNodes = kOctMomentNodes, kOmStr = kOmNodes + 2;  // LDS row stride: operand reads without bank conflicts

template <int L>
__global__ __launch_bounds__(256, 2) void k_oct_moments(const OctItem *items, const OctGroup *groups,
                                                         const double *PHI, double *part) {
    constexpr int NLM = (L + 1) * (L + 1), NS = kSlots<L>.n, NR = 2 * NLM;
    constexpr int NA = (NR * kOmNodes + 255) / 256;  // loads of H and U per thread
    __shared__ double X[8][16][kOmStr];              // [class][orbital][node]; the waves' sums at the end
    __shared__ double Y[NR + 1][kOmStr];             // rows of H, then of U, then zeros
    __shared__ short yrow[NS][16], qrow[NS][8];      // a slot's rows in Y; its harmonics (-1: none)
    const OctItem it = items[blockIdx.x];
    if (it.slot < 0) return;  // filler block
    const OctGroup gr = groups[it.group];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    for (int e = tid; e < NS * 8; e += 256) {
        int q = -1;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const int cl = kSlots<L>.cls[k], f = kSlots<L>.first[k];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (e == 8 * k + i && f + i < kCls<L>.count[cl]) q = kCls<L>.row[cl][f + i];
        }
        qrow[e >> 3][e & 7] = (short)q;
        yrow[e >> 3][e & 7] = (short)(q < 0 ? NR : q);
        yrow[e >> 3][8 + (e & 7)] = (short)(q < 0 ? NR : NLM + q);
    }
    if (tid < kOmStr) Y[NR][tid] = 0.0;
    const int nx = gr.nx, ny = gr.ny, nz = gr.nz;
    const int hx = (nx + 1) >> 1, hy = (ny + 1) >> 1, hz = (nz + 1) >> 1;
    const int Mo = hx * hy * hz;
    // loads: node tid % 32, orbitals tid / 32 and 8 + tid / 32 of the tile
    const int nd = tid & 31, o8 = tid >> 5;
    double f[2][8], y[NA];
    int dup = 0;
    auto load = [&](int t) {
        const int n = t * kOmNodes + nd, o = min(n, Mo - 1);
        int i, j, k;
        oct_coords(o, hx, hy, i, j, k);
        const int im = nx - 1 - i, jm = ny - 1 - j, km = nz - 1 - k;
        const int r00 = (k * ny + j) * nx, r01 = (k * ny + jm) * nx;
        const int r10 = (km * ny + j) * nx, r11 = (km * ny + jm) * nx;
        // an image on a centre plane is the node itself: once (bit 3: no node)
        dup = (i == im ? 1 : 0) | (j == jm ? 2 : 0) | (k == km ? 4 : 0) | (n < Mo ? 0 : 8);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double *P = PHI + gr.off + (long long)min(16 * it.ot0 + o8 + 8 * h, gr.n - 1) * gr.M;
            f[h][0] = P[r00 + i];
            f[h][1] = P[r00 + im];
            f[h][2] = P[r01 + i];
            f[h][3] = P[r01 + im];
            f[h][4] = P[r10 + i];
            f[h][5] = P[r10 + im];
            f[h][6] = P[r11 + i];
            f[h][7] = P[r11 + im];
        }
#pragma unroll
        for (int e = 0; e < NA; ++e) {
            const int r = min(o8 + 8 * e, NR - 1);
            y[e] = (r < NLM ? gr.H + (size_t)r * Mo : gr.U + (size_t)(r - NLM) * Mo)[o];
        }
    };
    dbl4 acc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) acc[k] = dbl4{0.0, 0.0, 0.0, 0.0};
    if (it.t0 < it.t1) load(it.t0);
    for (int t = it.t0; t < it.t1; ++t) {
        __syncthreads();  // the last tile's products are done (first: the tables)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool ook = 16 * it.ot0 + o8 + 8 * h < gr.n;
            double (&v)[8] = f[h];
#pragma unroll
            for (int m = 0; m < 8; ++m) v[m] = (ook && !((m | 8) & dup)) ? v[m] * v[m] : 0.0;
#pragma unroll
            for (int b = 1; b < 8; b <<= 1)
#pragma unroll
                for (int m = 0; m < 8; ++m)
                    if (!(m & b)) {
                        const double s = v[m] + v[m | b], d = v[m] - v[m | b];
                        v[m] = s;
                        v[m | b] = d;
                    }
#pragma unroll
            for (int m = 0; m < 8; ++m) X[m][o8 + 8 * h][nd] = v[m];
        }
#pragma unroll
        for (int e = 0; e < NA; ++e)
            if (o8 + 8 * e < NR) Y[o8 + 8 * e][nd] = y[e];
        if (t + 1 < it.t1) load(t + 1);
        lds_barrier();
#pragma unroll
        for (int s = 0; s < kOmNodes / 16; ++s) {
            const int n = 4 * (w + 4 * s) + g;
#pragma unroll
            for (int k = 0; k < NS; ++k) acc[k] = mfma(Y[yrow[k][c]][n], X[kSlots<L>.cls[k]][c][n], acc[k]);
        }
    }
    // the four waves' sums, added in order
    double *const out = part + gr.poff + (size_t)it.slot * gr.ot * 2 * NLM * 16;
    double *const sx = &X[0][0][0];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) sx[(4 * w + r) * 64 + lane] = acc[k][r];
        __syncthreads();
        const int rw = g + 4 * w, q = qrow[k][rw & 7];
        const double s = (sx[w * 64 + lane] + sx[(4 + w) * 64 + lane]) + (sx[(8 + w) * 64 + lane] + sx[(12 + w) * 64 + lane]);
        if (q >= 0) out[((size_t)(2 * it.ot0 + (rw >> 3)) * NLM + q) * 16 + c] = s;
    }
}

// The groups' partial sums added in block order, as operand fragments of
// k_sic_octant: frag[arr][tile][k step][lane], zero where a tile or a class
// ends early.  One block per (k step, tile, arr).
template <int L>
__global__ __launch_bounds__(1024) void k_oct_final(const OctTile *tiles, int ntiles, const double *part, double *frag) {
    constexpr int NLM = (L + 1) * (L + 1), KS = kSteps<L>;
    __shared__ double sx[16][64];
    const int ks = blockIdx.x, arr = blockIdx.z;
    const OctTile tl = tiles[blockIdx.y];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int g = lane >> 4, c = lane & 15;
    int q = -1;
#pragma unroll
    for (int cl = 0; cl < 8; ++cl)
        if (ks >= kCls<L>.ks[cl] && ks < kCls<L>.ks[cl + 1]) {
            const int i = 4 * (ks - kCls<L>.ks[cl]) + g;
            if (i < kCls<L>.count[cl]) q = kCls<L>.row[cl][i];
        }
    double s = 0.0;
    if (q >= 0 && c < tl.n) {
        const int go = tl.gorb + c;
        const double *p = part + tl.poff + ((size_t)(2 * (go >> 4) + arr) * NLM + q) * 16 + (go & 15);
        for (int b = w; b < tl.nparts; b += 16) s += p[(size_t)b * tl.ot * 2 * NLM * 16];
    }
    sx[w][lane] = s;
    __syncthreads();
    if (w == 0) {
        for (int k = 1; k < 16; ++k) s += sx[k][lane];
        frag[(((size_t)arr * ntiles + blockIdx.y) * KS + ks) * 64 + lane] = s;
    }
}

// ---------------------------------------------------------------------------
// Per node and orbital, from phi_i and w_i alone:
//   v_i = w_i + sum_q Q_q,i U_q,  rho_i = phi_i^2,  LSDA of rho_i,
//   sums of rho_i v_i and rho_i eps_xc (U_i, X_i), the Slater average V_SIC,
//   Gam_i = 2 dV phi_i omega_i, omega_i = -((v_i + A^T rho_i)/2 + v_xc,i),
//   written over w_i (the adjoint contraction's operand).
// A block takes 16 octant nodes at a time, its four waves the four mirror
// images in y and z; a wave walks the orbitals 16 at a time, and the products
// of the coefficient fragments with U and H (both in LDS) give both sums at
// its nodes and their x images.  Reads 16 B and writes 8 B per orbital node;
// bound by the LSDA's FP64 operations.  MODE 1: the fragments of all the group's
// orbitals fit in half the LDS; 2: in all of it, so one block of eight waves
// (two sets of 16 nodes) takes the compute unit; 0: they come 16 orbitals at
// a time.  With one mode of 256 threads for all, groups of three to six
// orbital tiles paid two more barriers a tile.  31 orbitals at 96^3: 263 us
// (the fields' bytes 130) where the boundary combination, the average, the
// adjoint field's expansion and source took 199 + 198 + 133 + 155; the
// descriptors in scalar registers and the unconditional prefetch are 17 of it.
// ---------------------------------------------------------------------------
template <int L, int MODE>
__global__ __launch_bounds__(MODE == 2 ? 512 : 256, 2) void k_sic_octant(
    const OctItem *__restrict__ items, const OctGroup *__restrict__ groups, const ChanDesc *__restrict__ chans,
    int ntiles, const double *__restrict__ frag, const double *__restrict__ PHI, double *W, double floor, int want_v,
    double *partU, double *partX) {
    constexpr int KS = kSteps<L>, NB = (2 * KS * 4 * 16 + 255) / 256;
    constexpr bool LF = MODE != 0;
    constexpr int SUB = MODE == 2 ? 2 : 1, NT = 256 * SUB, NW = 4 * SUB;
    extern __shared__ __attribute__((aligned(16))) double osm[];
    const OctItem *const ip = items + blockIdx.x;
    const OctItem it{uni(ip->group), 0, uni(ip->t0), uni(ip->t1), uni(ip->slot)};
    const OctGroup *const gp = groups + it.group;
    const int nx = uni(gp->nx), ny = uni(gp->ny), nz = uni(gp->nz), nchan = uni(gp->nchan), tile0 = uni(gp->tile0[0]);
    const int c0 = uni(gp->chan0);
    const int nt0 = (uni(chans[c0].N) + 15) >> 4;
    const int nt = nt0 + (nchan > 1 ? (uni(chans[c0 + 1].N) + 15) >> 4 : 0);  // fragment tiles of the group
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = w >> 2, t256 = tid & 255;
    double *const B = osm + sub * 2 * KS * 4 * 16;   // [2][4 KS][16]: U and H of these four waves' nodes
    double *const S = osm + SUB * 2 * KS * 4 * 16;   // [2][NW waves][16 nt]: sums of rho v and rho eps_xc
    double *const Fr = S + 2 * NW * 16 * nt;         // [2][nt (LF) or 1][KS][64]
    const int g = lane >> 4, c = lane & 15;
    const int ys = w & 1, zs = (w >> 1) & 1;
    const int hx = (nx + 1) >> 1, hy = (ny + 1) >> 1, hz = (nz + 1) >> 1;
    const int Mo = hx * hy * hz;
    for (int e = tid; e < 2 * NW * 16 * nt; e += NT) S[e] = 0.0;
    if (LF)
        for (int e = tid; e < 2 * nt * KS * 64; e += NT) {
            const int arr = e / (nt * KS * 64);
            Fr[e] = frag[((size_t)arr * ntiles + tile0) * KS * 64 + (e - arr * nt * KS * 64)];
        }
    __shared__ short qrow[4 * KS];  // harmonic of each operand row
    for (int e = tid; e < 4 * KS; e += NT) {
        int q = 0;
#pragma unroll
        for (int cl = 0; cl < 8; ++cl)
#pragma unroll
            for (int i = 0; i < 4 * (kCls<L>.ks[cl + 1] - kCls<L>.ks[cl]); ++i)
                if (e == 4 * kCls<L>.ks[cl] + i) q = kCls<L>.row[cl][i];
        qrow[e] = (short)q;
    }
    const double *const U = gp->U, *const H = gp->H;
    const ChanDesc &ch0 = chans[c0], &ch1 = chans[c0 + nchan - 1];
    const int N0 = uni(ch0.N), N1 = uni(ch1.N);
    const long long M = uni(gp->M), off0 = uni(ch0.off), off1 = uni(ch1.off);
    const double dV2 = 2.0 * ch0.h * ch0.h * ch0.h;
    // operand rows of the next nodes (16 rows a sweep, 16 nodes a row)
    double bn[NB];
    auto stage = [&](int t) {
        const int o = min(16 * (t + sub) + (tid & 15), Mo - 1);
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int r = min((t256 >> 4) + 16 * e, 8 * KS - 1), arr = r >= 4 * KS;
            bn[e] = (arr ? H : U)[(size_t)qrow[arr ? r - 4 * KS : r] * Mo + o];
        }
    };
    // this wave's image of node 16 t + c and that one's x image: offsets, and
    // whether they are nodes of their own (a centre plane's image is not)
    int i0 = 0, i1 = 0, n0 = 0, n1 = 0;
    bool in = false, in2 = false, inn = false, inn2 = false;
    auto place = [&](int t) {
        const int n = 16 * (t + sub) + c, o = min(n, Mo - 1);
        int i, j, k;
        oct_coords(o, hx, hy, i, j, k);
        const int im = nx - 1 - i, jw = ys ? ny - 1 - j : j, kw = zs ? nz - 1 - k : k;
        inn = n < Mo && t + sub < it.t1 && (!ys || jw != j) && (!zs || kw != k);
        inn2 = inn && i != im;
        const int rj = (kw * ny + jw) * nx;
        n0 = rj + i;
        n1 = rj + im;
    };
    // phi and w of the next 16 orbitals
    double pn[4][2] = {}, wn[4][2] = {};
    auto fields = [&](int tl) {
        const bool s = tl >= nt0;
        const int ot = s ? tl - nt0 : tl, N = s ? N1 : N0;
        const long long off = s ? off1 : off0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (16 * ot + 4 * r >= N) break;  // rows of four: none of these
            const long long a = off + (long long)min(16 * ot + g + 4 * r, N - 1) * M;
            pn[r][0] = PHI[a + n0];
            pn[r][1] = PHI[a + n1];
            wn[r][0] = W[a + n0];
            wn[r][1] = W[a + n1];
        }
    };
    // !LF: the next tile's fragments (LDS holds one tile's)
    double fn[LF ? 1 : NB];
    auto pieces = [&](int tl) {
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            const int x = min(tid + 256 * e, 2 * KS * 64 - 1), arr = x >= KS * 64;
            fn[LF ? 0 : e] = frag[((size_t)arr * ntiles + tile0 + tl) * KS * 64 + (x - arr * KS * 64)];
        }
    };
    __syncthreads();  // qrow, S and Fr
    if (it.t0 < it.t1) {
        if (!LF) pieces(0);
        place(it.t0);
        fields(0);
        stage(it.t0);
    }
    for (int t = it.t0; t < it.t1; t += SUB) {
        lds_barrier();  // the last nodes' operands are read
#pragma unroll
        for (int e = 0; e < NB; ++e)
            if (t256 + 256 * e < 2 * KS * 4 * 16) B[t256 + 256 * e] = bn[e];
        lds_barrier();
        stage(min(t + SUB, it.t1 - 1));
        i0 = n0;
        i1 = n1;
        in = inn;
        in2 = inn2;
        double num0 = 0.0, num1 = 0.0, den0 = 0.0, den1 = 0.0;
#pragma unroll 1
        for (int tl = 0; tl < nt; ++tl) {
            const bool sp = tl >= nt0;
            const int ot = sp ? tl - nt0 : tl, N = sp ? N1 : N0;
            const long long off = sp ? off1 : off0;
            double ph[4][2], wv[4][2];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    ph[r][m] = pn[r][m];
                    wv[r][m] = wn[r][m];
                }
            if (!LF) {
                lds_barrier();  // the last tile's fragments are read
#pragma unroll
                for (int e = 0; e < NB; ++e)
                    if (tid + 256 * e < 2 * KS * 64) Fr[tid + 256 * e] = fn[e];
                lds_barrier();
                pieces(tl + 1 < nt ? tl + 1 : 0);
            }
            // unconditional (past the last nodes: some nodes again): a load in a
            // branch ends in a copy, and a wait, where the branches meet
            if (tl + 1 == nt) place(t + SUB);
            fields(tl + 1 < nt ? tl + 1 : 0);
            // x-even (a[0]) and x-odd (a[1]) sums on this wave's side
            dbl4 aU[2], aH[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) aU[m] = aH[m] = dbl4{0.0, 0.0, 0.0, 0.0};
            const double *fu = Fr + (LF ? tl * KS * 64 : 0) + lane;
            const double *fh = fu + (LF ? nt : 1) * KS * 64;
#pragma unroll
            for (int cl = 0; cl < 8; ++cl) {
                const double sg = ((((cl >> 1) & ys) ^ ((cl >> 2) & zs)) & 1) ? -1.0 : 1.0;
#pragma unroll
                for (int ks = kCls<L>.ks[cl]; ks < kCls<L>.ks[cl + 1]; ++ks) {
                    const double u = B[(4 * ks + g) * 16 + c], h = B[(4 * KS + 4 * ks + g) * 16 + c];
                    aU[cl & 1] = mfma(fu[ks * 64], cl > 1 ? sg * u : u, aU[cl & 1]);
                    aH[cl & 1] = mfma(fh[ks * 64], cl > 1 ? sg * h : h, aH[cl & 1]);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (16 * ot + 4 * r >= N) break;
                const int orb = 16 * ot + g + 4 * r;
                const bool ok = orb < N;
                const double v0 = wv[r][0] + (aU[0][r] + aU[1][r]), v1 = wv[r][1] + (aU[0][r] - aU[1][r]);
                const double t0 = wv[r][0] + (aH[0][r] + aH[1][r]), t1 = wv[r][1] + (aH[0][r] - aH[1][r]);
                // (nodes and orbitals past the end have rho = 0)
                const double p0 = ok && in ? ph[r][0] : 0.0, p1 = ok && in2 ? ph[r][1] : 0.0;
                const double r0 = p0 * p0, r1 = p1 * p1;
                double ex0, ec0, vx0, vc0, ex1, ec1, vx1, vc1;
                lsda_pol(r0, floor, ex0, ec0, vx0, vc0);
                lsda_pol(r1, floor, ex1, ec1, vx1, vc1);
                const double x0 = vx0 + vc0, x1 = vx1 + vc1;
                double us = fma(r0, v0, r1 * v1), xs = fma(r0, ex0 + ec0, r1 * (ex1 + ec1));
                num0 = fma(-r0, v0 + x0, num0);
                num1 = fma(-r1, v1 + x1, num1);
                den0 += r0;
                den1 += r1;
                double *const Wr = W + (off + (long long)orb * M);
                if (ok && in) Wr[i0] = -dV2 * p0 * fma(0.5, v0 + t0, x0);
                if (ok && in2) Wr[i1] = -dV2 * p1 * fma(0.5, v1 + t1, x1);
                // over the 16 nodes; one lane per orbital adds to the wave's sums
                us = row_sum(us);
                xs = row_sum(xs);
                if (c == 0) {
                    S[w * 16 * nt + 16 * tl + g + 4 * r] += us;
                    S[(NW + w) * 16 * nt + 16 * tl + g + 4 * r] += xs;
                }
            }
            if (tl + 1 == nt0 || tl + 1 == nt) {  // the channel's last orbitals
                const ChanDesc &ch = sp ? ch1 : ch0;
                if (want_v && ch.vsic) {
#pragma unroll
                    for (int s = 16; s < 64; s <<= 1) {
                        num0 += __shfl_xor(num0, s, 64);
                        num1 += __shfl_xor(num1, s, 64);
                        den0 += __shfl_xor(den0, s, 64);
                        den1 += __shfl_xor(den1, s, 64);
                    }
                    if (g == 0 && in) ch.vsic[i0] = den0 > floor ? ch.vscale * num0 / den0 : 0.0;
                    if (g == 1 && in2) ch.vsic[i1] = den1 > floor ? ch.vscale * num1 / den1 : 0.0;
                }
                num0 = num1 = den0 = den1 = 0.0;
            }
        }
    }
    __syncthreads();
    int tl = 0;
    for (int cc = 0; cc < nchan; ++cc) {
        const ChanDesc &ch = chans[c0 + cc];
        const int N = ch.N, q = 16 * nt;
        for (int e = tid; e < N; e += NT) {
            const size_t p = (size_t)(ch.blk_base + it.slot) * kMaxOrb + e;
            const double *a = S + 16 * tl + e, *b = a + NW * q;
            double su = 0.0, sx = 0.0;
#pragma unroll
            for (int v = 0; v < NW; ++v) {
                su += a[v * q];
                sx += b[v * q];
            }
            partU[p] = su;
            partX[p] = sx;
        }
        tl += (N + 15) >> 4;
    }
}

// Uc = the first octant of nlm full-grid fields U
__global__ __launch_bounds__(256) void k_octant_pack(int nlm, int nx, int ny, int nz, const double *U, double *Uc) {
    const int hx = (nx + 1) / 2, hy = (ny + 1) / 2, hz = (nz + 1) / 2;
    const long long Mo = (long long)hx * hy * hz, M = (long long)nx * ny * nz;
    const long long n = (long long)nlm * Mo;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const long long q = e / Mo, o = e - q * Mo;
        const int i = (int)(o % hx), j = (int)((o / hx) % hy), k = (int)(o / ((long long)hx * hy));
        Uc[e] = U[q * M + ((long long)k * ny + j) * nx + i];
    }
}

hipError_t launch_octant_pack(int nlm, const int *n, const double *U, double *Uc, hipStream_t s) {
    if (nlm < 1 || nlm > kMaxLM || n[0] < 1 || n[1] < 1 || n[2] < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_octant_pack, dim3(1024), dim3(256), 0, s, nlm, n[0], n[1], n[2], U, Uc);
    return hipGetLastError();
}

#define FSIC_LMAX_SWITCH(lmax, F)                                                                          \
    switch (lmax) {                                                                                        \
        case 0: F(0); break;                                                                               \
        case 1: F(1); break;                                                                               \
        case 2: F(2); break;                                                                               \
        case 3: F(3); break;                                                                               \
        case 4: F(4); break;                                                                               \
        case 5: F(5); break;                                                                               \
        case 6: F(6); break;                                                                               \
        case 7: F(7); break;                                                                               \
        case 8: F(8); break;                                                                               \
        default: return hipErrorInvalidValue;                                                              \
    }

int oct_steps(int lmax) {
    static constexpr int ks[kMaxL + 1] = {kSteps<0>, kSteps<1>, kSteps<2>, kSteps<3>, kSteps<4>,
                                          kSteps<5>, kSteps<6>, kSteps<7>, kSteps<8>};
    return lmax >= 0 && lmax <= kMaxL ? ks[lmax] : 0;
}

hipError_t launch_oct_moments(int lmax, const OctItem *items, int nitems, const OctGroup *groups, const OctTile *tiles,
                              int ntiles, const double *PHI, double *part, double *frag, hipStream_t s) {
    if (nitems <= 0 || ntiles <= 0) return hipSuccess;
#define F(L)                                                                                                   \
    hipLaunchKernelGGL((k_oct_moments<L>), dim3(nitems), dim3(256), 0, s, items, groups, PHI, part);            \
    hipLaunchKernelGGL((k_oct_final<L>), dim3(kSteps<L>, ntiles, 2), dim3(1024), 0, s, tiles, ntiles, part, frag)
    FSIC_LMAX_SWITCH(lmax, F)
#undef F
    return hipGetLastError();
}

namespace {
// LDS bytes of the Slater step for groups of at most nt fragment tiles
size_t sic_lds(int lmax, int nt, int mode) {
    const size_t ks = (size_t)oct_steps(lmax), sub = mode == 2 ? 2 : 1;
    return (sub * 2 * ks * 4 * 16 + 2 * 4 * sub * 16 * (size_t)nt + 2 * (mode ? (size_t)nt : 1) * ks * 64) * sizeof(double);
}
// the statically allocated part, rounded up
constexpr size_t kSicStatic = 512;
int sic_mode(int lmax, int nt) {
    if (sic_lds(lmax, nt, 1) + kSicStatic <= 64 * 1024) return 1;
    return sic_lds(lmax, nt, 2) + kSicStatic <= 160 * 1024 ? 2 : 0;
}
template <int L>
const void *sic_kernel(int mode) {
    return mode == 0 ? (const void *)k_sic_octant<L, 0> : mode == 1 ? (const void *)k_sic_octant<L, 1>
                                                                    : (const void *)k_sic_octant<L, 2>;
}
}  // namespace

hipError_t launch_sic_octant(int lmax, const OctItem *items, int nitems, const OctGroup *groups, const ChanDesc *chans,
                             int ntiles, int group_tiles, const double *frag, const double *PHI, double *W,
                             double floor, int want_v, double *partU, double *partX, hipStream_t s) {
    if (nitems <= 0) return hipSuccess;
    const int mode = sic_mode(lmax, group_tiles);
    const size_t lds = sic_lds(lmax, group_tiles, mode);
#define GO(L, M) hipLaunchKernelGGL((k_sic_octant<L, M>), dim3(nitems), dim3(M == 2 ? 512 : 256), lds, s, items, groups, \
                                    chans, ntiles, frag, PHI, W, floor, want_v, partU, partX)
#define F(L)                                                                                             \
    if (const hipError_t e = allow_lds(sic_kernel<L>(mode), lds)) return e;                              \
    if (mode == 0) GO(L, 0);                                                                             \
    else if (mode == 1) GO(L, 1);                                                                        \
    else GO(L, 2)
    FSIC_LMAX_SWITCH(lmax, F)
#undef F
#undef GO
    return hipGetLastError();
}

int oct_slots(int kind, int lmax, int group_tiles) {
    static std::mutex mu;
    static std::map<std::array<int, 4>, int> cache;
    int dev = 0, cu = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || lmax < 0 || lmax > kMaxL) return 256;
    std::lock_guard<std::mutex> lk(mu);
    const std::array<int, 4> key{dev, kind, lmax, kind ? group_tiles : 0};
    const auto f = cache.find(key);
    if (f != cache.end()) return f->second;
    const int mode = kind ? sic_mode(lmax, group_tiles) : 0;
    const size_t lds = kind ? sic_lds(lmax, group_tiles, mode) : 0;
    const void *fn = nullptr;
#define F(L) fn = kind == 0 ? (const void *)k_oct_moments<L> : sic_kernel<L>(mode)
    switch (lmax) {
        case 0: F(0); break;
        case 1: F(1); break;
        case 2: F(2); break;
        case 3: F(3); break;
        case 4: F(4); break;
        case 5: F(5); break;
        case 6: F(6); break;
        case 7: F(7); break;
        default: F(8); break;
    }
#undef F
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu < 1) cu = 256;
    if (allow_lds(fn, lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, mode == 2 ? 512 : 256, lds) != hipSuccess || n < 1)
        n = 1;
    (void)hipGetLastError();  // a failed query leaves no error behind for the next launch
    return cache[key] = cu * n;
}

}  // namespace fsic
