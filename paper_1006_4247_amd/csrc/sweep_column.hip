// Register-resident sweeps for lattices around and beyond one workgroup's LDS: binary32
// L = 18 .. 32, binary64 L = 16 and 18.
//
// One workgroup owns one replica for the whole call.  Thread (g, q) owns the sites of both
// sublattices at place q = ih + (L/2) j of the planes z = g ZP .. g ZP + ZP - 1: their spins
// stay in its registers, so two of a site's neighbours along z are its own (other
// sublattice, same place, planes z - 1 and z + 1) and only those in the plane, and the
// ones beyond its run of planes, come from LDS.  HBM sees one read and one write of the
// replica per call, however many sweeps it makes, where the streaming kernels move three
// half-replicas per half-sweep.
//
// To L = 26, LDS holds one sublattice at a time, the one the current half-sweep reads: a
// half-sweep reads it, waits, and writes the updated sublattice over it.  The couplings
// along z stay in registers too; the other four of a site come from the L2 in every
// half-sweep, asked for two sites ahead.  Binary32 heat-bath half-sweeps draw the uniforms
// first, one Philox block per site pair, into LDS (where it has room for them).
//
// From L = 28, a sublattice is more than an LDS and the spins leave no registers for
// couplings (L = 32: 192 of a thread's 256).  A thread owns whole columns there (no plane
// is beyond its run), LDS holds BZ planes of a sublattice at a time in two buffers in
// turn, and all six couplings come from the L2.
//
// What bounds it (L = 24, 8 x 2 x 16 replicas, one per CU): an overrelaxation half-sweep
// takes 2.9 us, in which the VALU is 51 % and the LDS 47 % busy, the two only partly
// overlapping between the barriers of the one workgroup a CU holds (L = 28: 6.5 us, 41 and
// 39 %, two waves per SIMD).  1 heat-bath + 30 overrelaxation lattice sweeps of 8 x 2 x 27
// replicas: L = 24 0.42 ms, against 1.36 ms in 62 streaming launches at the rate of HBM;
// L = 28 0.88 against 2.16 ms; L = 32 1.02 against 2.71 ms.  A CU holds one replica, so
// that replicas beyond a multiple of 256 wait for a round of their own.
//
// Spins are those of the other sweep kernels bit for bit (same site arithmetic, order of
// the field's terms and random numbers), and so are the energies of sweeps where the size of
// an ensemble or the length of a call decides between this kernel and the streaming ones
// (column_energy).
#include "hsg_device.h"
#include "hsg_launch.h"

#include <cmath>
#include <type_traits>
#include <utility>

namespace hsg {

// ZP planes per run; WPE waves per SIMD the registers are budgeted for; SEL: the neighbour
// along x that is the thread's own is taken from its registers (two selects per component)
// instead of LDS; FENCE: bits 1, 2, 4 keep the compiler from mixing a site's loads with its
// arithmetic, a site with the next, two sites with the next two; bit 8 has threads without
// sites skip the writes to LDS that they otherwise repeat (the compiler spills less without
// the branch but at L = 26; all measured per size).  BZ, HZ: planes per buffer of an
// overrelaxation and of each half of a heat-bath half-sweep of whole columns.
template <typename T, int L>
struct ColumnShape;
template <int ZP_, int WPE_, bool SEL_, int FENCE_, int BZ_ = 0, int HZ_ = 0>
struct ColumnTuning {
    static constexpr int ZP = ZP_, WPE = WPE_, FENCE = FENCE_, BZ = BZ_, HZ = HZ_;
    static constexpr bool SEL = SEL_;
};
template <> struct ColumnShape<float, 18> : ColumnTuning<6, 4, true, 4> {};   // two workgroups per CU
template <> struct ColumnShape<float, 20> : ColumnTuning<4, 4, true, 4> {};
template <> struct ColumnShape<float, 22> : ColumnTuning<11, 2, false, 3> {};
template <> struct ColumnShape<float, 24> : ColumnTuning<8, 4, false, 3> {};
template <> struct ColumnShape<float, 26> : ColumnTuning<13, 3, false, 11> {};
template <> struct ColumnShape<float, 28> : ColumnTuning<28, 2, false, 3, 7, 7> {};
template <> struct ColumnShape<float, 30> : ColumnTuning<30, 2, false, 3, 5, 5> {};
template <> struct ColumnShape<float, 32> : ColumnTuning<32, 2, false, 3, 4, 4> {};
template <> struct ColumnShape<double, 16> : ColumnTuning<4, 2, false, 2> {};
template <> struct ColumnShape<double, 18> : ColumnTuning<6, 2, false, 3> {};

template <typename T, int L>
struct Column : ColumnShape<T, L> {
    static constexpr int ZP = ColumnShape<T, L>::ZP;
    static constexpr int HL = L / 2, PL = HL * L, NH = PL * L, N = 2 * NH, NQ = NH / 2;
    static constexpr int ZG = L / ZP;                      // runs of planes
    static constexpr int NT = ((PL * ZG + 63) / 64) * 64;  // threads
    static constexpr int B = static_cast<int>(sizeof(T));
    // LDS: one sublattice [3][NH], and the heat-bath uniforms [2][NH] of a half-sweep; or
    // (BZ > 0) two batches of BZ planes of a sublattice, [2][3][BZ PL]
    static constexpr int BZ = ColumnShape<T, L>::BZ, NB = BZ ? L / BZ : 1;
    static constexpr int CS = BZ ? BZ * PL : NH;  // from one component to the next
    static constexpr bool DRAWN = sizeof(T) == 4 && BZ == 0 && 5 * NH * 4 <= 150 * 1024;
    static constexpr bool JZ = BZ == 0;  // bonds along z in registers
    static constexpr int JN = JZ ? 4 : 6;
    static constexpr int HZ = ColumnShape<T, L>::HZ;  // planes of each half of the lattice per heat-bath step (BZ > 0)
    // the energy's site terms (see column_energy): their words over the site's uniforms, or
    // over the sublattice once it has been read, or (pairs of sites) beyond the batches
    static constexpr size_t TERMS = BZ      ? 6 * BZ * static_cast<size_t>(PL) * sizeof(T)
                                    : DRAWN ? 3 * static_cast<size_t>(NH) * sizeof(T)
                                            : 0;
    static constexpr size_t WAVES = DRAWN ? 0 : TERMS + (BZ ? NQ : NH) * 8;  // (the sublattice has been read)
    static constexpr int NG = (NQ + 63) / 64;  // waves of site pairs
    static constexpr bool TILED = !(sizeof(T) == 8 && L == 16);  // energies in the streaming kernels' order
    static constexpr size_t LDS = (BZ ? (12 * HZ + 12 > 6 * BZ ? 12 * HZ + 12 : 6 * BZ) * static_cast<size_t>(PL)
                                      : (DRAWN ? 5 : 3) * static_cast<size_t>(NH)) *
                                  sizeof(T);
    static_assert(L % ZP == 0 && ZP >= 2 && NT <= 1024, "one workgroup");
    static_assert(TERMS % 8 == 0 && WAVES % 8 == 0 && WAVES + NG * 8 <= LDS && NG <= 256, "room for the terms");
    static_assert(BZ == 0 || (ZG == 1 && L % BZ == 0 && NB % 2 == 0), "whole columns, batches in turn in two buffers");
};

__device__ __forceinline__ float buffer_get(__amdgpu_buffer_rsrc_t r, int voff, int soff, float) {
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ double buffer_get(__amdgpu_buffer_rsrc_t r, int voff, int soff, double) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return __hiloint2double(static_cast<int>(v.y), static_cast<int>(v.x));
}

// f(integral_constant m) for m = 0 .. N - 1, unrolled whatever the size of f.
template <class F, int... Ms>
__device__ __forceinline__ void each_plane_of(std::integer_sequence<int, Ms...>, F&& f) {
    (f(std::integral_constant<int, Ms>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void each_plane(F&& f) {
    each_plane_of(std::make_integer_sequence<int, N>{}, f);
}

// What a thread keeps for the whole call.
template <typename T, int L>
struct ColumnState {
    static constexpr int ZP = Column<T, L>::ZP;
    T s[2][ZP][3];    // spins [sublattice][plane of the run][component]
    T jb[2][Column<T, L>::JN];                 // couplings of the next two sites to update
    T jz[2][Column<T, L>::JZ ? ZP + 1 : 1];  // bonds along z: [sublattice of the lower end][plane - first plane + 1]
    // byte offsets of sites in a sublattice's array, in LDS and of the couplings alike: own
    // site of the run's first plane; [(P + m) & 1][+x, -x] (SEL: [..][2] is the one that is
    // not the thread's own); y neighbours; the planes below and above the run
    int own, x[2][3], yp, ym, zm, zp;
    // a thread without sites of its own (!on) repeats the last one's: it writes the same
    // values to the same places, and only its energies are left out
    bool on;
    bool o0;  // x = 2 ih + o with o = o0 where (P + m) is even
    __amdgpu_buffer_rsrc_t J;
    uint32_t g;
    int k0, k1;
};

// The couplings of the site of sublattice P in plane m of the run that registers do not hold.
template <typename T, int L, int P>
__device__ __forceinline__ void column_bonds(const ColumnState<T, L>& c, T (&j)[Column<T, L>::JN], int m, int so) {
    using M = Column<T, L>;
    constexpr int PL = M::PL, NH = M::NH, Q = 1 - P, B = M::B;
    // whole columns: two planes share a scalar offset, the second with an immediate one (six
    // scalar additions per two sites instead of twelve: L = 30, 1 + 30 lattice sweeps of 432
    // replicas 1080 -> 1025 us, L = 28 890 -> 876, L = 32 1033 -> 1021)
    const int me = M::BZ > 0 ? m & ~1 : m, im = (m - me) * PL * B;
    j[0] = buffer_get(c.J, c.own + im, so + (P * NH + me * PL) * B, T());
    j[1] = buffer_get(c.J, c.x[(P + m) & 1][1] + im, so + (Q * NH + me * PL) * B, T());
    j[2] = buffer_get(c.J, c.own + im, so + ((2 + P) * NH + me * PL) * B, T());
    j[3] = buffer_get(c.J, c.ym + im, so + ((2 + Q) * NH + me * PL) * B, T());
    if constexpr (!M::JZ) {
        const int md = m > 0 ? m - 1 : L - 1, mde = md & ~1;
        j[4] = buffer_get(c.J, c.own + im, so + ((4 + P) * NH + me * PL) * B, T());
        j[5] = buffer_get(c.J, c.own + (md - mde) * PL * B, so + ((4 + Q) * NH + mde * PL) * B, T());
    }
}

// Batch b (mod NB) of sublattice P into its buffer.
template <typename T, int L, int P>
__device__ __forceinline__ void column_publish(const ColumnState<T, L>& c, T* __restrict__ lds, int b) {
    using M = Column<T, L>;
#pragma unroll
    for (int k = 0; k < M::BZ; ++k)
#pragma unroll
        for (int mu = 0; mu < 3; ++mu)
            *reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(lds) + c.own +
                                  (((b & 1) * 3 + mu) * M::CS + k * M::PL) * M::B) = c.s[P][b * M::BZ + k][mu];
}

// One half-sweep of sublattice P: KIND 1 heat-bath, 2 overrelaxation, 3 overrelaxation
// with the energy, 0 general (kind, renormalisation and energy from the arguments).  The
// energy's terms are added up in `acc` (SUM) or left in LDS for column_energy, where nothing
// reads the sublattice or the uniforms after the call's last half-sweep.
template <typename T, int L, int P, int KIND, bool SUM>
__device__ __forceinline__ void column_half(ColumnState<T, L>& c, T* __restrict__ lds, bool hb_arg, bool rn_arg,
                                            bool want_arg, int hs, T beta, uint32_t tsw, double& acc, bool& bad) {
    using M = Column<T, L>;
    constexpr int PL = M::PL, NH = M::NH, NQ = M::NQ, ZP = M::ZP, NT = M::NT, Q = 1 - P, BZ = M::BZ;
    const bool hb = KIND == 0 ? hb_arg : KIND == 1;
    const bool rn = KIND == 0 && rn_arg;
    const bool want = KIND == 3 || (KIND == 0 && want_arg);
    // opaque copies keep the couplings' scalar offsets and the generator's key schedule inside
    // the half-sweep instead of letting them be hoisted and held in registers across the
    // kernel (no instruction emitted)
    int so = 0, k0 = __builtin_amdgcn_readfirstlane(c.k0), k1 = __builtin_amdgcn_readfirstlane(c.k1);
    asm volatile("" : "+s"(so), "+s"(k0), "+s"(k1));
    const auto at = [&](int off, int el) -> T& {  // LDS: byte offset of a thread + constant element
        return *reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(lds) + off + el * M::B);
    };
    double* const terms = reinterpret_cast<double*>(reinterpret_cast<unsigned char*>(lds) + M::TERMS) + c.own / M::B;
    constexpr bool HELD = !SUM && BZ == 0 && !M::DRAWN;  // terms in registers until the sublattice has been read
    double term[HELD ? ZP : 1];
    T* rnd = lds + 3 * NH;
    if (M::DRAWN && hb) {  // one Philox block per site pair (h, h + N/4)
        for (int h = static_cast<int>(threadIdx.x); h < NQ; h += NT) {
            const Words w = philox(static_cast<uint32_t>(h), tsw, c.g, heatbath_c3(hs), static_cast<uint32_t>(k0),
                                   static_cast<uint32_t>(k1));
            rnd[h] = static_cast<T>(u01_23(w.w0));
            rnd[NH + h] = static_cast<T>(u01_23(w.w1));
            rnd[NQ + h] = static_cast<T>(u01_23(w.w2));
            rnd[NH + NQ + h] = static_cast<T>(u01_23(w.w3));
        }
        lds_barrier();
    }
    each_plane<ZP>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        constexpr int e = (P + m) & 1;
        if constexpr (BZ > 0 && m % (BZ > 0 ? BZ : 1) == 0) {  // the next batch, which the barrier below completes
            if constexpr (m + BZ < ZP)
                column_publish<T, L, Q>(c, lds, m / (BZ > 0 ? BZ : 1) + 1);
            else
                column_publish<T, L, P>(c, lds, 0);  // (of the sublattice the next half-sweep reads)
        }
        T j[M::JN];
#pragma unroll
        for (int d = 0; d < M::JN; ++d) j[d] = c.jb[m & 1][d];
        T n[4][3], zlo[3], zhi[3];
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) {
            // the plane's place in LDS
            const int pl = BZ > 0 ? ((m / (BZ > 0 ? BZ : 1) & 1) * 3 + mu) * M::CS + m % (BZ > 0 ? BZ : 1) * PL
                                  : mu * NH + m * PL;
            if constexpr (M::SEL) {
                const T far = at(c.x[e][2], pl), near = c.s[Q][m][mu];
                const bool o = e ? !c.o0 : c.o0;
                n[0][mu] = o ? far : near;
                n[1][mu] = o ? near : far;
            } else {
                n[0][mu] = at(c.x[e][0], pl);
                n[1][mu] = at(c.x[e][1], pl);
            }
            n[2][mu] = at(c.yp, pl);
            n[3][mu] = at(c.ym, pl);
            if constexpr (M::ZG == 1) {
                zlo[mu] = c.s[Q][m > 0 ? m - 1 : ZP - 1][mu];
                zhi[mu] = c.s[Q][m + 1 < ZP ? m + 1 : 0][mu];
            } else {
                zlo[mu] = m > 0 ? c.s[Q][m > 0 ? m - 1 : 0][mu] : at(c.zm, mu * NH);
                zhi[mu] = m + 1 < ZP ? c.s[Q][m + 1 < ZP ? m + 1 : 0][mu] : at(c.zp, mu * NH);
            }
        }
        // the couplings of the site after next
        if constexpr (m + 2 < ZP) column_bonds<T, L, P>(c, c.jb[m & 1], m + 2, so);
        if (M::FENCE & 1) __builtin_amdgcn_sched_barrier(0);
        T S[3];
#pragma unroll
        for (int mu = 0; mu < 3; ++mu) {
            T v = T(0);
#pragma unroll
            for (int d = 0; d < 4; ++d) v = fma(j[d], n[d][mu], v);
            v = fma(M::JZ ? c.jz[P][M::JZ ? m + 1 : 0] : j[M::JN - 2], zhi[mu], v);
            v = fma(M::JZ ? c.jz[Q][M::JZ ? m : 0] : j[M::JN - 1], zlo[mu], v);
            S[mu] = v;
        }
        T ox, oy, oz;
        if (hb) {
            T r1, r2;
            int h = c.own / M::B + m * PL;
            if (!M::DRAWN) asm volatile("" : "+v"(h));  // the generator's first round stays in the half-sweep too
            if constexpr (M::DRAWN) {
                r1 = at(c.own, 3 * NH + m * PL);
                r2 = at(c.own, 4 * NH + m * PL);
            } else if constexpr (sizeof(T) == 4) {
                const bool hi = h >= NQ;
                const Words w = philox(static_cast<uint32_t>(hi ? h - NQ : h), tsw, c.g, heatbath_c3(hs),
                                       static_cast<uint32_t>(k0), static_cast<uint32_t>(k1));
                r1 = static_cast<T>(u01_23(hi ? w.w2 : w.w0));
                r2 = static_cast<T>(u01_23(hi ? w.w3 : w.w1));
            } else {
                const Words w = philox(static_cast<uint32_t>(h), tsw, c.g, heatbath_c3(hs), static_cast<uint32_t>(k0),
                                       static_cast<uint32_t>(k1));
                r1 = static_cast<T>(u01_52(w.w0, w.w1));
                r2 = static_cast<T>(u01_52(w.w2, w.w3));
            }
            heatbath<T>(S[0], S[1], S[2], beta, r1, r2, ox, oy, oz);
        } else {
            overrelax_flat<T>(c.s[P][m][0], c.s[P][m][1], c.s[P][m][2], S[0], S[1], S[2], ox, oy, oz);
            if (rn) renormalize(ox, oy, oz);
        }
        c.s[P][m][0] = ox;
        c.s[P][m][1] = oy;
        c.s[P][m][2] = oz;
        if (want) {
            const double dx = ox, dy = oy, dz = oz;
            double t = fma(dz, static_cast<double>(S[2]), fma(dy, static_cast<double>(S[1]), dx * static_cast<double>(S[0])));
            const double n2 = fma(dz, dz, fma(dy, dy, dx * dx));
            if (!(fabs(n2 - 1.0) <= NormTol<T>::value)) bad = true;
            if constexpr (SUM) {
                acc += t;
                asm volatile("" : "+v"(acc));  // or the sums are put off and every spin and field held for them
            } else if constexpr (BZ > 0) {  // planes m and m + L/2 are the thread's own
                if constexpr (m < ZP / 2)
                    terms[m * PL] = t;
                else
                    terms[(m - ZP / 2) * PL] += t;
            } else if constexpr (M::DRAWN) {
                const long long w = __double_as_longlong(t);
                at(c.own, 3 * NH + m * PL) = __int_as_float(static_cast<int>(w));
                at(c.own, 4 * NH + m * PL) = __int_as_float(static_cast<int>(w >> 32));
            } else {
                asm volatile("" : "+v"(t));  // (as above)
                term[m] = t;
            }
        }
        if ((M::FENCE & 2) || ((M::FENCE & 4) && (m & 1))) __builtin_amdgcn_sched_barrier(0);
        if (BZ > 0 && m % (BZ > 0 ? BZ : 1) == BZ - 1 && m + 1 < ZP) lds_barrier();
    });
    // the couplings of the next half-sweep's first two sites
    column_bonds<T, L, Q>(c, c.jb[0], 0, so);
    column_bonds<T, L, Q>(c, c.jb[1], 1, so);
    lds_barrier();  // every thread has read the other sublattice
    if constexpr (BZ == 0) {
        if (HELD && want) {
#pragma unroll
            for (int m = 0; m < ZP; ++m) terms[m * PL] = term[HELD ? m : 0];
        } else if ((M::FENCE & 8) == 0 || c.on) {
#pragma unroll
            for (int m = 0; m < ZP; ++m)
#pragma unroll
                for (int mu = 0; mu < 3; ++mu) at(c.own, mu * NH + m * PL) = c.s[P][m][mu];
        }
        lds_barrier();
    }
}

// The energy of the replica from the terms the call's last half-sweep left in LDS, in the
// order in which the streaming kernels add them (sites h and h + N/4, the wave butterfly,
// four waves of a 256-thread tile, the tiles): an ensemble's energies are then the same bits
// whichever of the two kernels takes a call, so that neither the size of an ensemble (a
// shard of it, say) nor the length of a call can change an exchange decision.  Every thread
// receives the result.
template <typename T, int L>
__device__ __forceinline__ double column_energy(T* __restrict__ lds, double& s_H) {
    using M = Column<T, L>;
    constexpr int NQ = M::NQ, NG = M::NG, NW = M::NT / 64, TILES = (NG + 3) / 4;
    static_assert(TILES <= 64, "a lane per tile");
    unsigned char* const raw = reinterpret_cast<unsigned char*>(lds);
    double* const waves = reinterpret_cast<double*>(raw + M::WAVES);
    const auto term = [&](int k) -> double {
        if constexpr (M::DRAWN) {
            const int* w = reinterpret_cast<const int*>(raw + M::TERMS);
            return __hiloint2double(w[M::NH + k], w[k]);
        }
        return reinterpret_cast<const double*>(raw + M::TERMS)[k];
    };
    const int lane = static_cast<int>(threadIdx.x) & 63, wave = static_cast<int>(threadIdx.x) >> 6;
#pragma unroll  // (the waves' sums interleave)
    for (int k = 0; k < (NG + NW - 1) / NW; ++k) {
        const int g = wave + k * NW, q = g * 64 + lane;
        double v = 0.0;
        if (q < NQ) v = M::BZ ? term(q) : term(q) + term(q + NQ);
        v = wave_sum(v);
        if (lane == 0 && g < NG) waves[g] = v;
    }
    lds_barrier();
    if (wave == 0) {
        double tile = 0.0, H = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if (4 * lane + w < NG) tile += waves[4 * lane + w];
#pragma unroll 4  // (more would spill scalar registers)
        for (int i = 0; i < TILES; ++i) H -= readlane_f64(tile, i);
        if (lane == 0) s_H = H;
    }
    lds_barrier();
    return s_H;
}

// A heat-bath half-sweep of sublattice P where a thread owns whole columns (BZ > 0).  Site
// pairs (h, h + N/4), L/2 planes apart, share a Philox block, so planes z and z + L/2 go
// together, HZ of each at a time: these planes of the other sublattice and the ones next
// to them go into LDS, the sites are then updated in a loop (one body instead of one per
// plane: unrolled like the overrelaxation it would not stay in the instruction cache), and
// their new spins return to the registers through LDS.
template <typename T, int L, int P>
__device__ __forceinline__ void column_heat(ColumnState<T, L>& c, T* __restrict__ lds, int hs, T beta, uint32_t tsw) {
    using M = Column<T, L>;
    constexpr int PL = M::PL, NH = M::NH, ZP = M::ZP, B = M::B, HZ = M::HZ, Q = 1 - P, HP = ZP / 2;
    static_assert(sizeof(T) == 4 && M::ZG == 1, "binary32 columns");
    int so = 0, k0 = __builtin_amdgcn_readfirstlane(c.k0), k1 = __builtin_amdgcn_readfirstlane(c.k1);
    asm volatile("" : "+s"(so), "+s"(k0), "+s"(k1));
    unsigned char* const raw = reinterpret_cast<unsigned char*>(lds);
    // [half][3][HZ + 2][PL] of sublattice Q, then [half][3][HZ][PL] new spins
    constexpr int CA = (HZ + 2) * PL * B, CN = HZ * PL * B, NEW = 6 * CA;
    const auto at = [&](int off) -> T& { return *reinterpret_cast<T*>(raw + off); };
    const auto bonds = [&](T (&j)[6], int m) {  // of plane m
        const int x1 = ((P + m) & 1) ? c.x[1][1] : c.x[0][1];
        const int z = m * PL * B, zd = (m > 0 ? m - 1 : L - 1) * PL * B;
        j[0] = buffer_get(c.J, c.own, so + P * NH * B + z, T());
        j[1] = buffer_get(c.J, x1, so + Q * NH * B + z, T());
        j[2] = buffer_get(c.J, c.own, so + (2 + P) * NH * B + z, T());
        j[3] = buffer_get(c.J, c.ym, so + (2 + Q) * NH * B + z, T());
        j[4] = buffer_get(c.J, c.own, so + (4 + P) * NH * B + z, T());
        j[5] = buffer_get(c.J, c.own, so + (4 + Q) * NH * B + zd, T());
    };
    each_plane<HP / HZ>([&](auto bc) __attribute__((always_inline)) {
        constexpr int z0 = decltype(bc)::value * HZ;
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int k = 0; k < HZ + 2; ++k)
#pragma unroll
                for (int mu = 0; mu < 3; ++mu)
                    at(c.own + (half * 3 + mu) * CA + k * PL * B) = c.s[Q][(z0 + half * HP + k - 1 + ZP) % ZP][mu];
        T jn[2][6];
        bonds(jn[0], z0);
        bonds(jn[1], z0 + HP);
        lds_barrier();
#pragma unroll 1
        for (int k = 0; k < HZ; ++k) {
            T j[2][6];
#pragma unroll
            for (int half = 0; half < 2; ++half)
#pragma unroll
                for (int d = 0; d < 6; ++d) j[half][d] = jn[half][d];
            if (k + 1 < HZ) {
                bonds(jn[0], z0 + k + 1);
                bonds(jn[1], z0 + k + 1 + HP);
            }
            const Words w = philox(static_cast<uint32_t>(c.own / B + (z0 + k) * PL), tsw, c.g, heatbath_c3(hs),
                                   static_cast<uint32_t>(k0), static_cast<uint32_t>(k1));
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int odd = (P + z0 + k + half * HP) & 1;
                const int xp = odd ? c.x[1][0] : c.x[0][0], xm = odd ? c.x[1][1] : c.x[0][1];
                const int pl = half * 3 * CA + (k + 1) * PL * B;
                const int nb[6] = {xp + pl, xm + pl, c.yp + pl, c.ym + pl, c.own + pl + PL * B, c.own + pl - PL * B};
                T S[3] = {T(0), T(0), T(0)}, o[3];
#pragma unroll
                for (int d = 0; d < 6; ++d)
#pragma unroll
                    for (int mu = 0; mu < 3; ++mu) S[mu] = fma(j[half][d], at(nb[d] + mu * CA), S[mu]);
                heatbath<T>(S[0], S[1], S[2], beta, static_cast<T>(u01_23(half ? w.w2 : w.w0)),
                            static_cast<T>(u01_23(half ? w.w3 : w.w1)), o[0], o[1], o[2]);
#pragma unroll
                for (int mu = 0; mu < 3; ++mu) at(NEW + c.own + (half * 3 + mu) * CN + k * PL * B) = o[mu];
            }
        }
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int k = 0; k < HZ; ++k)
#pragma unroll
                for (int mu = 0; mu < 3; ++mu)
                    c.s[P][z0 + half * HP + k][mu] = at(NEW + c.own + (half * 3 + mu) * CN + k * PL * B);
        lds_barrier();  // the planes have been read
    });
    // the couplings and the batch the next half-sweep starts with
    column_bonds<T, L, Q>(c, c.jb[0], 0, so);
    column_bonds<T, L, Q>(c, c.jb[1], 1, so);
    column_publish<T, L, P>(c, lds, 0);
    lds_barrier();
}

// One sweep: n_hb heat-bath then n_or overrelaxation lattice sweeps, sublattice 0 before 1,
// or (ADJ) in reverse.  The loops over kinds are separate so that the spins a thread holds
// stay in place from one half-sweep to the next.
template <typename T, int L, bool SUM, bool ADJ>
__device__ __forceinline__ void column_sweep(ColumnState<T, L>& c, T* __restrict__ lds, int n_hb, int n_or, bool renorm,
                                             bool want, T beta, uint32_t tsw, double& acc, bool& bad) {
    constexpr int P0 = ADJ ? 1 : 0, P1 = 1 - P0;
    const int n_lat = n_hb + n_or;
    if constexpr (Column<T, L>::BZ > 0) {  // n_hb > 0 and n_or > 0 (column_faster)
        static_assert(!ADJ, "no legs on whole columns");
        for (int l = 0; l < n_hb; ++l) {
            column_heat<T, L, 0>(c, lds, 2 * l, beta, tsw);
            column_heat<T, L, 1>(c, lds, 2 * l + 1, beta, tsw);
        }
        for (int l = want ? 1 : 0; l < n_or; ++l) {
            column_half<T, L, 0, 2, SUM>(c, lds, false, false, false, 0, beta, tsw, acc, bad);
            column_half<T, L, 1, 2, SUM>(c, lds, false, false, false, 0, beta, tsw, acc, bad);
        }
        if (want) {
            column_half<T, L, 0, 2, SUM>(c, lds, false, false, false, 0, beta, tsw, acc, bad);
            column_half<T, L, 1, 3, SUM>(c, lds, false, false, true, 0, beta, tsw, acc, bad);
        }
        return;
    }
    // the lattice sweep that renormalises (the last overrelaxation one of the forward order,
    // where there is no heat-bath) or ends with the energy runs in the general form
    const int head = ADJ && renorm ? 1 : 0, tail = (want || (renorm && !ADJ)) && !(head && n_lat == 1) ? 1 : 0;
    const auto general = [&](int i) {  // i-th lattice sweep of the call's order
        const int l = ADJ ? n_lat - 1 - i : i;
        const bool hb = l < n_hb, rn = renorm && l == n_lat - 1, w = want && i == n_lat - 1;
        column_half<T, L, P0, 0, SUM>(c, lds, hb, rn, false, 2 * l + P0, beta, tsw, acc, bad);
        column_half<T, L, P1, 0, SUM>(c, lds, hb, rn, w, 2 * l + P1, beta, tsw, acc, bad);
    };
    const auto heat = [&](int i0, int i1) {
        for (int i = i0; i < i1; ++i) {
            const int l = ADJ ? n_lat - 1 - i : i;
            column_half<T, L, P0, 1, SUM>(c, lds, true, false, false, 2 * l + P0, beta, tsw, acc, bad);
            column_half<T, L, P1, 1, SUM>(c, lds, true, false, false, 2 * l + P1, beta, tsw, acc, bad);
        }
    };
    const auto over = [&](int i0, int i1) {
        for (int i = i0; i < i1; ++i) {
            column_half<T, L, P0, 2, SUM>(c, lds, false, false, false, 0, beta, tsw, acc, bad);
            column_half<T, L, P1, 2, SUM>(c, lds, false, false, false, 0, beta, tsw, acc, bad);
        }
    };
    const int end = n_lat - tail;
    if constexpr (!ADJ) {
        heat(0, n_hb < end ? n_hb : end);
        over(n_hb < end ? n_hb : end, end);
        if (tail && n_or > 0 && !renorm) {
            column_half<T, L, P0, 2, SUM>(c, lds, false, false, false, 0, beta, tsw, acc, bad);
            column_half<T, L, P1, 3, SUM>(c, lds, false, false, true, 0, beta, tsw, acc, bad);
        } else if (tail) {
            general(end);
        }
    } else {
        if (head) general(0);
        over(head, n_or < end ? n_or : end);
        heat(n_or < end ? n_or : end, end);
        if (tail) general(end);
    }
}

struct ColumnLeg {  // an annealing leg's protocol
    double a, b;
    const double* tab;
    int K;
    __device__ __forceinline__ double lam(int k) const {  // point k = 0 .. K + 1, ascending for the up-leg
        if (k <= 0) return a;
        if (k >= K + 1) return b;
        return tab ? tab[k - 1] : a + static_cast<double>(k) * (b - a) / static_cast<double>(K + 1);
    }
};

// The sweeps of one replica: from `gs`, through n_sweeps sweeps (LEG: the leg's K sweeps at
// its protocol points, ADJ in adjoint order), to `gd`.  Returns the final energy; W is the
// leg's work.
template <typename T, int L, bool LEG, bool ADJ, class Src>
__device__ __forceinline__ double column_run(const hsg_ensemble& e, int slot, Src gs, T* gd, int n_sweeps,
                                             int n_hb, int n_or, const ColumnLeg& leg, double H, double& W,
                                             unsigned char* smem_raw, double* red, double& s_H) {
    using M = Column<T, L>;
    constexpr int HL = M::HL, PL = M::PL, NH = M::NH, N = M::N, NT = M::NT, ZP = M::ZP, B = M::B;
    T* lds = reinterpret_cast<T*>(smem_raw);
    const int tid = static_cast<int>(threadIdx.x);
    const int R = e.n_temps;
    const T* J = static_cast<const T*>(e.couplings) + static_cast<size_t>(slot / (e.n_chains * R)) * 3 * N;
    const uint32_t t0 = e.sweep_ctr[slot];
    ColumnState<T, L> c;
    c.J = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(J), 0, 3 * N * B, 0x00027000);
    c.g = e.slot_base + static_cast<uint32_t>(slot);
    c.k0 = static_cast<int>(key_lo(e.seed));
    c.k1 = static_cast<int>(key_hi(e.seed));
    c.on = tid < PL * M::ZG;
    {
        const int t = c.on ? tid : PL * M::ZG - 1;
        const int zg = t / PL, q = t - zg * PL;
        const int j = q / HL, ih = q - j * HL;
        const int z0 = zg * ZP, base = z0 * PL;
        const int q_xp = j * HL + (ih + 1 == HL ? 0 : ih + 1), q_xm = j * HL + (ih == 0 ? HL - 1 : ih - 1);
        const int q_yp = (j + 1 == L ? 0 : j + 1) * HL + ih, q_ym = (j == 0 ? L - 1 : j - 1) * HL + ih;
        c.own = (base + q) * B;
        c.o0 = (j + z0) & 1;
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int o = v ^ ((j + z0) & 1);
            c.x[v][0] = (base + (o ? q_xp : q)) * B;
            c.x[v][1] = (base + (o ? q : q_xm)) * B;
            c.x[v][2] = (base + (o ? q_xp : q_xm)) * B;
        }
        c.yp = (base + q_yp) * B;
        c.ym = (base + q_ym) * B;
        c.zm = ((z0 == 0 ? L - 1 : z0 - 1) * PL + q) * B;
        c.zp = ((z0 + ZP == L ? 0 : z0 + ZP) * PL + q) * B;
    }
    const int own = c.own / B;
    // a sweep that opens with a heat-bath half-sweep of parity 0 reads no parity-0 spin
    const bool skip0 = n_hb > 0 && !ADJ;
    const auto load = [&](int p) {
#pragma unroll
        for (int m = 0; m < ZP; ++m)
#pragma unroll
            for (int mu = 0; mu < 3; ++mu) c.s[p][m][mu] = gs[(mu * 2 + p) * NH + own + m * PL];
    };
    load(1);
    if (!skip0) {
        load(0);
    } else {
#pragma unroll
        for (int m = 0; m < ZP; ++m) c.s[0][m][0] = c.s[0][m][1] = c.s[0][m][2] = T(0);
    }
    if constexpr (M::JZ)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        c.jz[p][0] = J[(4 + p) * NH + c.zm / B];
#pragma unroll
        for (int m = 0; m < ZP; ++m) c.jz[p][m + 1] = J[(4 + p) * NH + own + m * PL];
    }
    constexpr int FIRST = ADJ ? 1 : 0;  // the sublattice updated first
    column_bonds<T, L, FIRST>(c, c.jb[0], 0, 0);
    column_bonds<T, L, FIRST>(c, c.jb[1], 1, 0);
    if constexpr (M::BZ > 0) {
        column_publish<T, L, 1 - FIRST>(c, lds, 0);
    } else {
#pragma unroll
        for (int m = 0; m < ZP; ++m)
#pragma unroll
            for (int mu = 0; mu < 3; ++mu) lds[mu * NH + own + m * PL] = c.s[1 - FIRST][m][mu];
    }
    lds_barrier();

    const bool renorm = renorm_on(e) && n_hb == 0;
    const int n_iter = LEG ? leg.K + 1 : n_sweeps;
    bool bad = false;
    constexpr bool SUM = LEG || !M::TILED;
    for (int k = 0; k < n_iter; ++k) {
        double beta_d;
        if (LEG) {
            const double cur = ADJ ? leg.lam(leg.K + 1 - k) : leg.lam(k);
            beta_d = ADJ ? leg.lam(leg.K - k) : leg.lam(k + 1);
            W += (beta_d - cur) * H;
            if (k == leg.K) break;
        } else {
            beta_d = e.betas[label(e.temp_of_slot[slot], R, e.guard)];
        }
        const bool need_e = LEG || k == n_sweeps - 1;
        double acc = 0.0;
        column_sweep<T, L, SUM, ADJ>(c, lds, n_hb, n_or, renorm, need_e, static_cast<T>(beta_d), t0 + static_cast<uint32_t>(k),
                                acc, bad);
        if (SUM && need_e) {
            const double tot = block_sum<NT, true>(c.on ? acc : 0.0, red);
            if (tid == 0) s_H = -tot;
            lds_barrier();
            H = s_H;
        }
    }
    if (c.on) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int m = 0; m < ZP; ++m)
#pragma unroll
                for (int mu = 0; mu < 3; ++mu) gd[(mu * 2 + p) * NH + own + m * PL] = c.s[p][m][mu];
    }
    if constexpr (!SUM) H = column_energy<T, L>(lds, s_H);  // (the spins need no registers any more)
    if (bad || !isfinite(H)) atomicOr(e.guard, 1);
    if (tid == 0) e.sweep_ctr[slot] = t0 + static_cast<uint32_t>(LEG ? leg.K : n_sweeps);
    return H;
}

// Regular sweeps, one workgroup per replica.
template <typename T, int L>
__global__ void __launch_bounds__((Column<T, L>::NT), (Column<T, L>::WPE))
    k_column(hsg_ensemble e, int n_sweeps, int n_hb, int n_or) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[Column<T, L>::NT / 64];
    __shared__ double s_H;
    const int slot = xcd_order(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
    T* gs = static_cast<T*>(e.spins) + static_cast<size_t>(slot) * 3 * Column<T, L>::N;
    double W = 0.0;
    const double H = column_run<T, L, false, false, const T*>(e, slot, gs, gs, n_sweeps, n_hb, n_or, ColumnLeg{}, 0.0, W, smem_raw,
                                                    red, s_H);
    if (threadIdx.x == 0) e.energy[slot] = H;
}

// Annealing legs of the pairs i = parity (mod 2), one workgroup per (chain, pair, leg),
// from the spins into the candidate buffer.
template <typename T, int L>
__global__ void __launch_bounds__((Column<T, L>::NT), (Column<T, L>::WPE))
    k_column_leg(hsg_ensemble e, int n_hb, int n_or, int parity) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[Column<T, L>::NT / 64];
    __shared__ double s_H;
    constexpr int N = Column<T, L>::N;
    const int R = e.n_temps;
    const int bid = xcd_order(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
    const int npp = (R - parity) / 2;
    const int down = bid & 1, rest = bid >> 1, ch = rest / npp;
    const int ipair = parity + 2 * (rest % npp);
    const int slot = ch * R + label(e.slot_of_temp[ch * R + ipair + down], R, e.guard);
    ColumnLeg leg;
    leg.K = e.anneal_K[ipair];
    if (leg.K < 0 || leg.K > e.anneal_K_max) {
        if (threadIdx.x == 0) atomicOr(e.guard, 2);
        leg.K = leg.K < 0 ? 0 : e.anneal_K_max;
    }
    leg.a = e.betas[ipair];
    leg.b = e.betas[ipair + 1];
    leg.tab = e.anneal_lambda ? e.anneal_lambda + static_cast<size_t>(ipair) * e.anneal_K_max : nullptr;
    const ScratchLayout sl = scratch_layout(e);
    unsigned char* scr = static_cast<unsigned char*>(e.scratch);
    double H = e.energy[slot], W = 0.0;
    using Src = const T* __restrict__;  // (source and destination of a leg are two arrays, a replica's are one)
    const T* gs = static_cast<const T*>(e.spins) + static_cast<size_t>(slot) * 3 * N;
    T* gd = reinterpret_cast<T*>(scr + sl.cand) + static_cast<size_t>(slot) * 3 * N;
    if (leg.K == 0)
        W = down ? (leg.a - leg.b) * H : (leg.b - leg.a) * H;
    else if (down)
        H = column_run<T, L, true, true, Src>(e, slot, gs, gd, 0, n_hb, n_or, leg, H, W, smem_raw, red, s_H);
    else
        H = column_run<T, L, true, false, Src>(e, slot, gs, gd, 0, n_hb, n_or, leg, H, W, smem_raw, red, s_H);
    if (threadIdx.x == 0) {
        e.work[(static_cast<size_t>(ch) * (R - 1) + ipair) * 2 + down] = W;
        reinterpret_cast<double*>(scr + sl.cand_energy)[slot] = H;
    }
}

template <typename T, int L>
static hipError_t go_column(const hsg_ensemble& e, int n_sweeps, int n_hb, int n_or, hipStream_t st) {
    using M = Column<T, L>;
    auto kern = k_column<T, L>;
    const hipError_t err = allow_dynamic_lds(reinterpret_cast<const void*>(kern), M::LDS);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(e.n_samples * e.n_chains * e.n_temps), dim3(M::NT), M::LDS, st, e, n_sweeps, n_hb, n_or);
    return hipGetLastError();
}

template <typename T, int L>
static hipError_t go_column_legs(const hsg_ensemble& e, int parity, int n_hb, int n_or, hipStream_t st) {
    using M = Column<T, L>;
    const int blocks = e.n_samples * e.n_chains * ((e.n_temps - parity) / 2) * 2;
    if (blocks <= 0) return hipSuccess;
    auto kern = k_column_leg<T, L>;
    const hipError_t err = allow_dynamic_lds(reinterpret_cast<const void*>(kern), M::LDS);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(M::NT), M::LDS, st, e, n_hb, n_or, parity);
    return hipGetLastError();
}

// Binary32 L = 18 .. 32 and binary64 L = 16, 18: where the registers and LDS of a CU hold
// the replica (beyond, a thread's spins alone exceed its registers).
bool column_supported(const hsg_ensemble& e) {
    if (max_block_lds() < 160 * 1024) return false;
    if (e.precision == HSG_FP64) return e.L == 16 || e.L == 18;
    return e.L >= 18 && e.L <= 32 && (e.L & 1) == 0;
}

// ... and where it is the faster kernel.  The streaming kernels pay per half-sweep, with a
// launch and, once the replicas fill it, at the rate of HBM; this one pays once for bringing a
// replica in and out, then per lattice sweep, a heat-bath one two to four times an
// overrelaxation (more from L = 26, where the uniforms have no room in LDS), and its time
// hardly depends on the replicas up to one per CU.  So it loses few replicas, few lattice
// sweeps and many heat-baths.  Both times in us from fits to 2385 measured calls, 4 .. 432
// slots and 1 .. 124 lattice sweeps in 20 compositions: the rule takes the slower kernel by
// more than 3 % in 8 of them on this side and 35 on the other, all near the line (the worst
// 44 / 39 us and 41 / 34).  Column / streaming in us at 32, 96, 256 and 432 slots: binary32
// L = 18, 1 + 0: 14 / 12, 15 / 17, 17 / 23, 23 / 31; L = 22, 1 + 0: 21 / 16, 22 / 21, 24 / 34,
// 46 / 48; L = 24, 1 + 3: 45 / 42, 46 / 66, 56 / 127, 102 / 182, 1 + 30: 202 / 289, 202 / 474,
// 212 / 933, 413 / 1344; L = 26, 1 + 3: 68 / 55, 76 / 83, 90 / 165, 167 / 250, 1 + 30: 291 /
// 362, 300 / 573, 316 / 1229, 619 / 1864; L = 32, 1 + 3: 103 / 54, 105 / 108, 119 / 223, 226 /
// 362, 1 + 30: 499 / 380, 499 / 795, 518 / 1664, 1027 / 2679; binary64 L = 18, 1 + 3: 48 / 50,
// 49 / 76, 56 / 131, 105 / 209.  Binary64 L = 16 against the LDS-resident kernel, 6 .. 432
// slots: 1 + 0 22 / 24 .. 46 / 61, 1 + 30 106 / 148 .. 217 / 305.
struct ColumnCost {
    float in_out, per_slot, hb, over;             // this kernel, a round of 256 replicas
    float sweep, half_min, half_0, half_slot;     // streaming: per sweep, per lattice sweep
};
static ColumnCost column_cost(const hsg_ensemble& e) {
    if (e.precision == HSG_FP64) return {11.4f, 0.031f, 23.9f, 4.1f, 3.8f, 12.8f, 7.5f, 0.091f};
    switch (e.L) {
        case 18: return {6.5f, 0.012f, 7.6f, 3.0f, 4.0f, 8.9f, 7.7f, 0.039f};
        case 20: return {6.4f, 0.013f, 8.3f, 3.1f, 3.4f, 8.7f, 6.9f, 0.056f};
        case 22: return {8.6f, 0.016f, 12.5f, 4.2f, 4.7f, 9.2f, 7.6f, 0.077f};
        case 24: return {9.6f, 0.034f, 15.7f, 5.9f, 5.0f, 8.8f, 6.6f, 0.089f};
        case 26: return {11.5f, 0.063f, 26.1f, 8.8f, 7.0f, 8.1f, 8.0f, 0.121f};
        case 28: return {10.1f, 0.042f, 38.5f, 12.8f, 7.0f, 8.6f, 7.6f, 0.143f};
        case 30: return {10.8f, 0.053f, 44.1f, 15.2f, 7.4f, 8.8f, 8.2f, 0.179f};
        default: return {11.7f, 0.063f, 44.3f, 14.8f, 6.5f, 8.3f, 6.1f, 0.189f};
    }
}

// fused: the streaming sweeps' last finishing launch is the measurement's (launch_measure_fin).
bool column_faster(const hsg_ensemble& e, int n_sweeps, int n_hb, int n_or, bool fused) {
    if (!column_supported(e)) return false;
    const bool f64 = e.precision == HSG_FP64;
    if (f64 && e.L == 16) return true;
    // (whole columns neither renormalise nor take the energy after a heat-bath)
    if (e.L > 26 && (n_hb == 0 || n_or == 0)) return false;
    const ColumnCost c = column_cost(e);
    const float n = static_cast<float>(n_sweeps), slots = static_cast<float>(e.n_samples) * e.n_chains * e.n_temps;
    const float once = c.in_out + n * (n_hb * c.hb + n_or * c.over);
    float column;
    if (!f64 && e.L == 18)  // two replicas per CU
        column = (once + c.per_slot * std::fmin(slots, 256.0f)) * std::fmax(1.0f, std::ceil(slots / 256.0f) * 0.75f);
    else
        column = once * std::ceil(slots / 256.0f) + c.per_slot * slots;
    // (workgroups in a number that is no multiple of the XCDs are not ordered by them: xcd_order)
    const long long tiles = (static_cast<long long>(e.L) * e.L * e.L / 4 + 255) / 256;
    const bool ordered = tiles * e.n_samples * e.n_chains * e.n_temps % 8 == 0;
    const float half = std::fmax(c.half_min, c.half_0 + c.half_slot * slots * (ordered ? 1.0f : 1.5f));
    const float stream = n * (c.sweep + (n_hb * (f64 ? 1.3f : 1.05f) + n_or) * half) - (fused ? c.sweep : 0.0f);
    return column <= (!f64 && e.L <= 22 ? 1.0f : 0.97f) * stream;
}

hipError_t launch_column_sweeps(const hsg_ensemble& e, int n_sweeps, int n_hb, int n_or, hipStream_t st) {
    if (e.precision == HSG_FP64)
        return e.L == 16 ? go_column<double, 16>(e, n_sweeps, n_hb, n_or, st)
                         : go_column<double, 18>(e, n_sweeps, n_hb, n_or, st);
    switch (e.L) {
        case 18: return go_column<float, 18>(e, n_sweeps, n_hb, n_or, st);
        case 20: return go_column<float, 20>(e, n_sweeps, n_hb, n_or, st);
        case 22: return go_column<float, 22>(e, n_sweeps, n_hb, n_or, st);
        case 24: return go_column<float, 24>(e, n_sweeps, n_hb, n_or, st);
        case 26: return go_column<float, 26>(e, n_sweeps, n_hb, n_or, st);
        case 28: return go_column<float, 28>(e, n_sweeps, n_hb, n_or, st);
        case 30: return go_column<float, 30>(e, n_sweeps, n_hb, n_or, st);
        default: return go_column<float, 32>(e, n_sweeps, n_hb, n_or, st);
    }
}

// Annealing legs: where this kernel is not the slower one for any number of legs.  The choice
// does not depend on that number, as the two kernels add the energies of a leg in different
// orders and its work decides the exchange: a shard of an ensemble has to take the decisions
// of the whole.  A leg takes its energy in every sweep and holds more than a replica's sweeps
// do, so few legs with many heat-baths stream sooner.  Column / streaming, us a call, K = 8,
// 2 and 416 legs: binary32 L = 22, 1 + 0: 151 / 145, 335 / 471, 1 + 3: 257 / 380, 547 / 1424;
// L = 24, 1 + 1: 266 / 223, 640 / 862 (streams), 1 + 3: 358 / 371, 821 / 1569; L = 26, 1 + 3: 594
// / 391, 1487 / 2065 (streams); binary64 L = 18, 1 + 0: 382 / 208, 859 / 591 (streams), 1 + 3: 401
// / 577, 888 / 1732.  (Binary64 L = 16: k_resident_leg.)
bool column_legs_faster(const hsg_ensemble& e, int n_hb, int n_or) {
    if (!column_supported(e) || e.L <= 16 || e.L > 24) return false;
    if (e.precision == HSG_FP32 && e.L <= 22) return true;
    return n_or >= 2 && n_or >= 3 * n_hb;
}

hipError_t launch_column_legs(const hsg_ensemble& e, int parity, int n_hb, int n_or, hipStream_t st) {
    if (e.precision == HSG_FP64) return go_column_legs<double, 18>(e, parity, n_hb, n_or, st);
    switch (e.L) {
        case 18: return go_column_legs<float, 18>(e, parity, n_hb, n_or, st);
        case 20: return go_column_legs<float, 20>(e, parity, n_hb, n_or, st);
        case 22: return go_column_legs<float, 22>(e, parity, n_hb, n_or, st);
        case 24: return go_column_legs<float, 24>(e, parity, n_hb, n_or, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace hsg
