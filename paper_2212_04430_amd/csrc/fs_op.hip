// The shifted Wilson-Dirac operator on canonical spinors, without a block layout.
//
// fs_apply_dirac used to copy the spinors, convert them to the solver's block
// layout, run the stencil there, convert back and copy out: five passes over
// the fields besides the stencil's own, and for small lattices ten launches and
// table uploads.  Here a workgroup owns a TX x TY x TZ tile of one spinor's sites
// and walks t, reading complex128 spinors as they lie ([site][12], 192 bytes)
// and writing the result the same way.
//
// * The slice's spinors, rounded to the storage precision, sit in LDS; lanes
//   inside the tile find their neighbours there, only lanes on a face read them
//   from memory.  The forward-t neighbour of slice t is the LDS entry of t + 1,
//   the backward-t term is carried in registers.
// * Tiles need not divide the lattice (lanes beyond its end idle), so odd
//   extents take the same kernel.
// * The spinors of one tile are consecutive workgroups, so they find the links
//   in the XCD's L2.
//
// Bound: memory (in and out once, links once) and, at two to three waves per SIMD,
// its latency for large lattices; one slice's latency for small ones.  Measured
// per call, block layout -> here: 4^4 FP64 97 -> 24 us, 9x7x5x11 FP32 with three
// spinors 102 -> 24, 16^3x32 FP32 with twelve 702 -> 223 (2.9 TB/s), 32^3x64 FP64
// 1363 -> 478 (4.2 TB/s).
#include "fs_stencil.h"
#include "fs_op.h"

namespace fs {

namespace {

// Canonical spinors lie 192 bytes apart, so one 16-byte load per lane of its own
// spinor touches 64 lines, twelve times over: the address unit was 80% busy.
// Lanes of a quad therefore move their four spinors together, 64 bytes of one
// spinor per instruction, and exchange the pieces with DPP moves.

// 4 x 4 transposition over a quad: lane j gives e[k], k = 0..3, and receives the
// e[j] of lane k in e[k].
__device__ __forceinline__ void quad_transpose(uint32_t e[4]) {
    const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
#pragma unroll
    for (int k = 0; k < 4; k += 2) {  // lanes j and j ^ 1: quad_perm 1 0 3 2
        const uint32_t send = odd ? e[k] : e[k + 1];
        const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0xB1, 0xF, 0xF, false);
        e[k] = odd ? got : e[k];
        e[k + 1] = odd ? e[k + 1] : got;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {  // lanes j and j ^ 2: quad_perm 2 3 0 1
        const uint32_t send = high ? e[k] : e[k + 2];
        const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send, 0x4E, 0xF, 0xF, false);
        e[k] = high ? got : e[k];
        e[k + 2] = high ? e[k + 2] : got;
    }
}

// The same for four complex numbers per lane.
__device__ __forceinline__ void quad_transpose(float re[4], float im[4]) {
    uint32_t a[4], b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        a[k] = __float_as_uint(re[k]);
        b[k] = __float_as_uint(im[k]);
    }
    quad_transpose(a);
    quad_transpose(b);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        re[k] = __uint_as_float(a[k]);
        im[k] = __uint_as_float(b[k]);
    }
}
__device__ __forceinline__ void quad_transpose(double re[4], double im[4]) {
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        double* const v = part ? im : re;
        uint32_t lo[4], hi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            lo[k] = (uint32_t)__double2loint(v[k]);
            hi[k] = (uint32_t)__double2hiint(v[k]);
        }
        quad_transpose(lo);
        quad_transpose(hi);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = __hiloint2double((int)hi[k], (int)lo[k]);
    }
}

// Forms the values here: without it the compiler moves the arithmetic behind them
// into the conditional stores, with every operand kept live (up to 2.6 KB per
// lane of spills).
template <typename A>
__device__ __forceinline__ void pin(A v[24]) {
#pragma unroll
    for (int k = 0; k < 24; ++k) asm volatile("" : "+v"(v[k]));
}

// The spinor at `site` in A.  Every lane of the quad takes part.
template <typename A>
__device__ __forceinline__ void load_canonical(const double2* __restrict__ in, int site, A v[24]) {
    const int qd = threadIdx.x & 3;
    const double2* p[4] = {in + (size_t)quad_bcast<0>(site) * 12 + qd, in + (size_t)quad_bcast<1>(site) * 12 + qd,
                           in + (size_t)quad_bcast<2>(site) * 12 + qd, in + (size_t)quad_bcast<3>(site) * 12 + qd};
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        A re[4], im[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double2 d = p[k][4 * m];
            re[k] = (A)d.x;
            im[k] = (A)d.y;
        }
        quad_transpose(re, im);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[8 * m + 2 * k] = re[k];
            v[8 * m + 2 * k + 1] = im[k];
        }
    }
    pin(v);
}

// The same rounded to storage precision P, in the form the hops take.
template <int P>
__device__ __forceinline__ void load_in(const double2* __restrict__ in, int site, typename PairIn<P>::T& x) {
    load_canonical<typename Tr<P>::acc>(in, site, x.v);
    round_sp<P, typename Tr<P>::acc>(x.v);
}

// Stores the spinors of the quad's valid lanes, rounded to storage precision P.
template <int P, typename A>
__device__ __forceinline__ void store_canonical(double2* __restrict__ out, int site, bool valid, A v[24]) {
    round_sp<P, A>(v);
    pin(v);
    const int qd = threadIdx.x & 3;
    const int w = valid ? site : -1;
    const int sk[4] = {(int)quad_bcast<0>(w), (int)quad_bcast<1>(w), (int)quad_bcast<2>(w), (int)quad_bcast<3>(w)};
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        A re[4], im[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            re[k] = v[8 * m + 2 * k];
            im[k] = v[8 * m + 2 * k + 1];
        }
        quad_transpose(re, im);
#pragma unroll
        for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(re[k]), "+v"(im[k]));
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (sk[k] >= 0) out[(size_t)sk[k] * 12 + 4 * m + qd] = make_double2((double)re[k], (double)im[k]);
    }
}

// One neighbour: the LDS entry nl when it is inside the tile, else the spinor at
// `site`.  Every lane issues the load (those inside the tile all of site 0, a
// broadcast) and the value is selected: any branch here, also a wave-uniform one,
// makes the compiler keep all hops' operands live (572 to 1276 bytes of spills).
template <int P>
__device__ __forceinline__ void op_fetch(bool inside, const double2* __restrict__ in, int site, const char* sh, int wg,
                                         int nl, typename PairIn<P>::T& x) {
    typename PairIn<P>::T g, l;
    load_in<P>(in, inside ? 0 : site, g);
    in_get<P>(sh, wg, nl, l);
    in_sel<P>(inside, l, g, x);
}

// Both hops along one spatial axis: lattice coordinate c of extent L (site stride
// ss), tile coordinate i of extent T (lane stride ls).  SPAN: the tile spans the
// axis, so every neighbour is inside it; else `whole` says so at run time.
template <int P, int Q, int MU, bool SPAN, typename PF, typename PB>
__device__ __forceinline__ void op_axis(const LatDesc& ld, const double2* __restrict__ in, const char* sh, int wg,
                                        int lane, int site, int c, int L, int ss, int i, int T, int ls,
                                        typename Tr<P>::acc o[24]) {
    using A = typename Tr<P>::acc;
    const bool whole = T == L;
    typename PairIn<P>::T x;
    {
        const bool end = c == L - 1;
        const int sf = end ? site - (L - 1) * ss : site + ss;
        const bool inside = SPAN || (end ? whole : i < T - 1);
        const int nl = !inside ? lane : end ? lane - (L - 1) * ls : lane + ls;
        if constexpr (SPAN) in_get<P>(sh, wg, nl, x);
        else op_fetch<P>(inside, in, sf, sh, wg, nl, x);
        hop_fwd<P, Q, PF>(ld, MU, site, x, o, A(-0.5));
    }
    {
        const bool end = c == 0;
        const int sb = end ? site + (L - 1) * ss : site - ss;
        const bool inside = SPAN || (end ? whole : i > 0);
        const int nl = !inside ? lane : end ? lane + (L - 1) * ls : lane - ls;
        if constexpr (SPAN) in_get<P>(sh, wg, nl, x);
        else op_fetch<P>(inside, in, sb, sh, wg, nl, x);
        hop_bwd<P, Q, PB>(ld, MU, sb, x, o, A(-0.5));
    }
}

// Resident waves per SIMD to compile for: FP64 keeps about 240 registers live.
template <int P> struct OpW { static constexpr int v = P == P64 ? 2 : 3; };

// SX: the tile spans x.  Lanes beyond the tile or the lattice compute a clamped
// site and store nothing (the quad exchanges need every lane).  Q: link loads (0,
// or 3 where FP32 calls of four or more spinors rebuild row 2 of special unitary
// links).  Each term is formed and added in the order of k_dslash (diagonal, t, x,
// y, z), so in reduced storage, where another order would differ in the last
// stored bits, both give the same values.  (FP16 stays with k_dslash: the scale
// products in its t hops are fused into the projections or not depending on the
// slice's place in a chunk, which no other kernel repeats.)  FP64 takes t last: one LDS buffer,
// and the next slice's spinor lives only from there to the end of the slice.
template <int P, int Q, bool SX>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OpW<P>::v, 8)))
k_op(OpPlan a, LatDesc ld, double diag, const double2* __restrict__ in0, double2* __restrict__ out0) {
    using A = typename Tr<P>::acc;
    using In = typename PairIn<P>::T;
    constexpr int LB = in_lds_bytes<P>();
    constexpr bool TWO = tile_nbuf<P>() == 2;
    extern __shared__ uint4 lds_dyn[];
    char* const shb = reinterpret_cast<char*>(lds_dyn);
    const int wg = blockDim.x, lane = threadIdx.x;
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    if (id >= a.n_wg) return;
    const int rhs = id % a.n_rhs;
    int q = id / a.n_rhs;
    const int jx = q % a.nt[0];
    q /= a.nt[0];
    const int jy = q % a.nt[1];
    q /= a.nt[1];
    const int jz = q % a.nt[2], ch = q / a.nt[2];
    const int Lx = ld.L[0], Ly = ld.L[1], Lz = ld.L[2], Lt = ld.L[3];
    const int t0 = ch * a.tc, t1 = min(Lt, t0 + a.tc);
    const int ix = lane % a.T[0];
    q = lane / a.T[0];
    const int iy = q % a.T[1], iz = q / a.T[1];
    int x = jx * a.T[0] + ix, y = jy * a.T[1] + iy, z = jz * a.T[2] + iz;
    const bool valid = iz < a.T[2] && x < Lx && y < Ly && z < Lz;
    if (!valid) x = y = z = 0;
    const int sy = Lx, sz = Lx * Ly, st = sz * Lz;
    const int xyz = x + sy * y + sz * z;
    const double2* const in = in0 + (size_t)rhs * ld.V * 12;
    double2* const out = out0 + (size_t)rhs * ld.V * 12;
    A bw[12];
    {
        In e;
        A h[12], u[18];
        load_in<P>(in, xyz + st * t0, e);
        in_put<P>(shb, wg, lane, e);
        const int sb = xyz + st * (t0 == 0 ? Lt - 1 : t0 - 1);
        load_in<P>(in, sb, e);
        PtP::project(e.v, h);
        link<P, Q, A>(ld, 3, sb, u);
        mul_udag(u, h, bw);
        if (t0 == 0 && ld.tsign < 0) {
#pragma unroll
            for (int k = 0; k < 12; ++k) bw[k] = -bw[k];
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
        const char* const sh = shb + (TWO ? ((t - t0) & 1) : 0) * LB * wg;      // slice t
        char* const shn = shb + (TWO ? ((t - t0 + 1) & 1) : 0) * LB * wg;       // slice t + 1
        const int site = xyz + st * t;
        const bool wrap = t == Lt - 1;
        In nx;
        A o[24];
        // the diagonal and both t hops; the centre gives the backward-t term of
        // slice t + 1, the next slice's spinor the forward hop, by the same link
        auto hop_t = [&] {
            A u[18], h[12], w[12], bn[12];
            load_in<P>(in, wrap ? xyz : site + st, nx);
            link<P, Q, A>(ld, 3, site, u);
            {
                In c;
                in_get<P>(sh, wg, lane, c);
#pragma unroll
                for (int k = 0; k < 24; ++k) o[k] = TWO ? (A)diag * c.v[k] : fma_((A)diag, c.v[k], o[k]);
                PtP::project(c.v, h);
                mul_udag(u, h, TWO ? bn : bw);
            }
            PtM::project(nx.v, h);
            mul_u(u, h, w);
            PtM::accum(o, w, (wrap && ld.tsign < 0) ? A(0.5) : A(-0.5));
            if (TWO) {
                in_put<P>(shn, wg, lane, nx);
                PtP::accum(o, bw, A(-0.5));
#pragma unroll
                for (int k = 0; k < 12; ++k) bw[k] = bn[k];
            }
        };
        if constexpr (TWO) {
            hop_t();
        } else {
#pragma unroll
            for (int k = 0; k < 24; ++k) o[k] = A(0);
            PtP::accum(o, bw, A(-0.5));
        }
        // scheduling barriers keep each axis's loads in its own phase:
        // hoisted together they overflow the register file
        __builtin_amdgcn_sched_barrier(0);
        op_axis<P, Q, 0, SX, PxM, PxP>(ld, in, sh, wg, lane, site, x, Lx, 1, valid ? ix : 0, a.T[0], 1, o);
        __builtin_amdgcn_sched_barrier(0);
        op_axis<P, Q, 1, false, PyM, PyP>(ld, in, sh, wg, lane, site, y, Ly, sy, valid ? iy : 0, a.T[1], a.T[0], o);
        __builtin_amdgcn_sched_barrier(0);
        op_axis<P, Q, 2, false, PzM, PzP>(ld, in, sh, wg, lane, site, z, Lz, sz, valid ? iz : 0, a.T[2],
                                          a.T[0] * a.T[1], o);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!TWO) hop_t();
        store_canonical<P, A>(out, site, valid, o);
        if (t + 1 < t1) {
            __syncthreads();  // every read of slice t ends before its buffer is written
            if constexpr (!TWO) {
                in_put<P>(shn, wg, lane, nx);
                __syncthreads();
            }
        }
    }
}

}  // namespace

// Tile of at most `lanes` sites: the fewest spinor loads and lane slots.  Per
// lane of a workgroup and slice: its own spinor in and out and its links (about
// 3 spinors' worth), and on each face one neighbour from memory.
static void op_tile(const int* L, int lanes, int T[3]) {
    double best = 1e300;
    for (int c = 1; c <= std::min(L[2], lanes); ++c)
        for (int b = 1; b <= std::min(L[1], lanes / c); ++b) {
            const int a = std::min(L[0], lanes / (b * c));
            // the same number of tiles along x with even extents
            const int nx = (L[0] + a - 1) / a, ax = (L[0] + nx - 1) / nx;
            const double tiles = (double)nx * ((L[1] + b - 1) / b) * ((L[2] + c - 1) / c);
            const double faces = (ax < L[0] ? 2.0 / ax : 0.0) + (b < L[1] ? 2.0 / b : 0.0) + (c < L[2] ? 2.0 / c : 0.0);
            // a tile that spans x issues no x loads at all
            const double cost = tiles * lanes * (ax < L[0] ? 3.5 : 3.0) + (double)L[0] * L[1] * L[2] * faces;
            if (cost < best * (1.0 - 1e-9)) {
                best = cost;
                T[0] = ax;
                T[1] = b;
                T[2] = c;
            }
        }
}

OpPlan op_plan(int prec, const int* L, int n_rhs, bool two_rows) {
    OpPlan p;
    p.two_rows = two_rows;
    const long long V = (long long)L[0] * L[1] * L[2] * L[3];
    // workgroups of one wave spread a small problem over more CUs
    p.lanes = V * n_rhs >= (1 << 17) ? 256 : 64;
    op_tile(L, p.lanes, p.T);
    long long tiles = 1;
    for (int k = 0; k < 3; ++k) {
        p.nt[k] = (L[k] + p.T[k] - 1) / p.T[k];
        tiles *= p.nt[k];
    }
    // chunks of t: each costs two more spinor loads per lane, and the workgroups
    // run in rounds of the resident ones (of 256 lanes per CU: two in FP64, else
    // three, by registers)
    const double R = 256.0 * (prec == P64 ? 2 : 3) * (256 / p.lanes);
    double best = 1e300;
    p.tc = L[3];
    for (int nch = 1; nch <= L[3]; ++nch) {
        const int tc = (L[3] + nch - 1) / nch;
        const double wgs = (double)tiles * n_rhs * ((L[3] + tc - 1) / tc);
        const double cost = std::ceil(wgs / R) * (tc + 0.6);
        if (cost < best * (1.0 - 1e-9)) {
            best = cost;
            p.tc = tc;
        }
    }
    p.n_rhs = n_rhs;
    p.n_wg = tiles * n_rhs * ((L[3] + p.tc - 1) / p.tc);
    return p;
}

void launch_op(int prec, const OpPlan& p, const LatDesc& ld, double diag, const double* in, double* out,
               hipStream_t s) {
    const dim3 grid((unsigned)((p.n_wg + 7) / 8 * 8)), wg(p.lanes);
    const double2* i2 = reinterpret_cast<const double2*>(in);
    double2* o2 = reinterpret_cast<double2*>(out);
    const size_t lds = (size_t)p.lanes * (prec == P64 ? tile_nbuf<P64>() * in_lds_bytes<P64>()
                                                      : tile_nbuf<P32>() * in_lds_bytes<P32>());
    const bool sx = p.T[0] == ld.L[0];
#define FS_OP(PP, QQ)                                                                                 \
    if (sx) hipLaunchKernelGGL((k_op<PP, QQ, true>), grid, wg, lds, s, p, ld, diag, i2, o2);          \
    else hipLaunchKernelGGL((k_op<PP, QQ, false>), grid, wg, lds, s, p, ld, diag, i2, o2);            \
    break;
    switch (prec) {
        case P64: FS_OP(P64, 0)
        case P32:
            if (p.two_rows) {
                FS_OP(P32, 3)
            }
            FS_OP(P32, 0)
        case PBF: FS_OP(PBF, 0)
        default: break;
    }
#undef FS_OP
}

}  // namespace fs
