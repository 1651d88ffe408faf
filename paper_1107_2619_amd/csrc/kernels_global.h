// Global-gather density and force kernels and their dispatch, one translation
// unit per precision and species count (kernels_global_*.hip).  Data layout (all
// in the caller-provided workspace, see md_runtime.hip):
//   - atoms live in "slots" sorted by link cell (paper, "OpenMP
//     Parallelisation": particles ordered by link-cell index so cell members
//     are contiguous); replica r owns a wavefront-aligned slot range;
//   - positions as double4 {x, y, z, F'}: one 32-byte gather per neighbour
//     brings the position and the embedding derivative the force pass needs;
//   - the Verlet list is one int32 row per atom (slot index + periodic shift
//     code), read four entries per 16-byte load;
//   - the full (symmetric) list lets each atom gather its own density and
//     force with no atomics; the half list with FP64 atomics is kept as the
//     comparison variant (paper, "OpenMP Parallelisation", on the trade
//     between a symmetric list and synchronised updates).
#pragma once

#include "md_device.h"

namespace mdk {
namespace {
// Pair separation from compact records.  With the cell offset dc in {-1,0,1}
// per axis, d_a = (q_j - q_i + dc 2^28) h_a 2^-28: the integer part is exact
// in 32 bits (|d| < 8 cells), and the scale is one rounding in FP64.  `qi1`
// holds q_i + 2^28, so the field c = dc + 1 of the entry adds c 2^28.
__device__ __forceinline__ double compact_axis(int code_field, int qj, int qi1, double qs)
{
    const uint32_t dq = ((uint32_t)code_field << kCompactBits) + (uint32_t)qj - (uint32_t)qi1;
    return (double)(int32_t)dq * qs;
}

// CMP = 1: orthorhombic cells.  CMP = 2: a sheared cell, whose records hold
// fractional in-cell coordinates: the integer differences along the three edge
// vectors map through qg = h diag(2^-28 / n_a) into the Cartesian separation.
template <int CMP>
__device__ __forceinline__ void compact_delta(const DevReplica& R, const int4& qi1, const int4& qj, int code,
                                              double& dx, double& dy, double& dz)
{
    if (CMP == 2) {
        const double d0 = compact_axis(code & 3, qj.x, qi1.x, 1.0);
        const double d1 = compact_axis((code >> 2) & 3, qj.y, qi1.y, 1.0);
        const double d2 = compact_axis((code >> 4) & 3, qj.z, qi1.z, 1.0);
        dx = fma(R.qg[0], d0, fma(R.qg[1], d1, R.qg[2] * d2));
        dy = fma(R.qg[3], d0, fma(R.qg[4], d1, R.qg[5] * d2));
        dz = fma(R.qg[6], d0, fma(R.qg[7], d1, R.qg[8] * d2));
        return;
    }
    dx = compact_axis(code & 3, qj.x, qi1.x, R.qs[0]);
    dy = compact_axis((code >> 2) & 3, qj.y, qi1.y, R.qs[1]);
    dz = compact_axis((code >> 4) & 3, qj.z, qi1.z, R.qs[2]);
}

__device__ __forceinline__ int4 compact_base(const int4& q)
{
    constexpr int one = 1 << kCompactBits;
    return make_int4(q.x + one, q.y + one, q.z + one, q.w);
}

// One 16-byte gather through a raw buffer resource: a single load
// instruction with a 32-bit offset (out-of-range offsets read zero).
typedef int int4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t record_rsrc(const int4* p, int64_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int4*>(p), (short)0, (int)(n * 16), (int)kBufferWord3);
}
__device__ __forceinline__ int4 record_load(__amdgpu_buffer_rsrc_t rs, int j)
{
    const int4v v = __builtin_amdgcn_raw_buffer_load_b128(rs, j * 16, 0, 0);
    return make_int4(v.x, v.y, v.z, v.w);
}

// ---------------------------------------------------------------------------
// Global-gather kernels: every atom's neighbours straight from the cache
// hierarchy through the transposed int32 list.  Neighbours go in groups of
// kChunk = 4 (one 16-byte list load): all index loads, then all gathers, then
// the arithmetic.  Entries past the end point at the atom itself (masked).
//
// Every sum over neighbours is taken group by group: the four terms of a group
// in order, then the group's sum onto the atom's.  A group's sum does not
// depend on who computes it, so the two forms below give the same bits:
//   - k_density, k_force: one thread per atom walks its groups;
//   - k_density_split, k_force_split: the groups of 64 atoms are dealt to the
//     waves of a workgroup.
//
// FP64 mode reads a 32-byte {x, y, z, F'} record per neighbour, from LDS where it
// is one of the workgroup's own slots (Stage), the compact mixed mode a 16-byte
// record from the caches.
//
// NCH: neighbour records in flight per thread (2, 4 or 8; the autotuner picks
// it): more hide more gather latency, fewer free registers for more waves.
//
// The compact mixed mode reads its list groups one round ahead (AHEAD), behind the
// records of the round before, so that a round waits for one load and not for two
// in a row; its registers allow it (58 of the 64 for eight waves).  Step times
// without and with: 218,972 atoms 48.8 -> 47.5 us, 427,680 atoms 70.4 -> 69.9,
// 1,013,760 atoms 160.0 -> 158.3, 48 two-species replicas of 8,100 atoms
// 123.4 -> 121.0.  The FP64 mode loses (218,972 atoms 58.3 -> 60.6): it already
// has twice the bytes in flight, and four registers more cost it a wave.
//
// TL: several species with all their tables staged in LDS, in workgroups of
// kTableBlock threads that share one copy (one species always stages its own).

// The FP64 records of a workgroup's own slots, staged in LDS, where 63% of a
// crystal's neighbours lie (256 slots; 70% of 512): the L1 resolves one lane's
// 16-byte access per clock and CU, and an FP64 record takes two, which bound the
// force pass (74% of its time); from LDS a record costs a quarter of that.  Step
// times, from the caches against staged: 218,972 atoms 59.8 and 60.7 us, 278,404
// atoms 71.4 -> 67.3, 427,680 atoms 96.3 -> 88.2, 1,013,760 atoms 183.6 -> 162.6
// (force 98 -> 86, density 61 -> 52).  Below four wavefronts per SIMD latency
// binds and staging adds to it (KernelShape::stage).  The 16-byte compact records
// of mixed precision gain nothing (1,013,760 atoms 163 us either way): there the
// vector units are as busy as the L1; nor do several species, whose workgroups of
// 1024 hold all tables (1,024,000 atoms 258 us either way).  Workgroups of 512 do
// as well at 1,013,760 atoms (165.5 us) and worse at 427,680 (99, the last round
// of workgroups).
//
// Beside large tables the staged records would cost more than they save: they are
// staged where the LDS of a CU still holds four workgroups of the force pass, or six
// of the density pass, whose registers allow more (kStageLds).  Steps of 1,013,760
// atoms, from the caches and staged, by the LDS of the staged force pass: 18 KB 185 ->
// 164 us, 24 KB 191 -> 175, 28 KB 191 -> 173, 34 KB (energies) 234 -> 230; 40.2 KB 195
// and 207, 41.2 KB (energies) 230 and 243, 59 KB (energies) 258 and 297; density
// alone: 26 KB 195 -> 191, 32 KB 214 and 218.
//
// The two halves of a record lie in separate arrays, so that a random 16-byte read
// may fall on any bank.  FULL: with F' (the force pass).
//
// The staged records are read through LDS pointers (address space 3): through
// plain ones the compiler may merge a lane's LDS and global read into one flat
// load, which costs the whole gain.
typedef double double2v __attribute__((ext_vector_type(2)));

template <bool FULL>
constexpr size_t kStageLds = 160 * 1024 / (FULL ? 4 : 6);

template <bool FULL>
struct Stage {
    __attribute__((address_space(3))) unsigned char* mem;
    int t0;
    static constexpr size_t kBytes = kBlock * (FULL ? 32 : 24);
    __device__ __forceinline__ Stage(unsigned char* m, int first)
        : mem((__attribute__((address_space(3))) unsigned char*)m), t0(first)
    {
    }
    __device__ __forceinline__ __attribute__((address_space(3))) double2v* xy() const
    {
        return (__attribute__((address_space(3))) double2v*)mem;
    }
    __device__ __forceinline__ __attribute__((address_space(3))) double2v* zf() const { return xy() + kBlock; }
    __device__ __forceinline__ __attribute__((address_space(3))) double* zs() const
    {
        return (__attribute__((address_space(3))) double*)(mem + 16 * kBlock);
    }
    __device__ __forceinline__ void put(unsigned l, const double3& x) const
    {
        xy()[l] = (double2v){x.x, x.y};
        zs()[l] = x.z;
    }
    __device__ __forceinline__ void put(unsigned l, const double4& x) const
    {
        xy()[l] = (double2v){x.x, x.y};
        zf()[l] = (double2v){x.z, x.w};
    }
    // the record of staged slot t0 + l
    __device__ __forceinline__ void get(unsigned l, double3& x) const
    {
        const double2v a = xy()[l];
        x = make_double3(a.x, a.y, zs()[l]);
    }
    __device__ __forceinline__ void get(unsigned l, double4& x) const
    {
        const double2v a = xy()[l], c = zf()[l];
        x = make_double4(a.x, a.y, c.x, c.y);
    }
    static __device__ __forceinline__ void load(const double4* pos, int j, double3& x) { x = load_xyz(pos, j); }
    static __device__ __forceinline__ void load(const double4* pos, int j, double4& x) { x = pos[j]; }
    // The records of entries e: all LDS reads (some record for the lanes whose
    // neighbour is not staged), then the other lanes' loads.
    template <bool STAGE, int NCH, typename V>
    __device__ __forceinline__ void gather(const double4* pos, const int (&e)[NCH], V (&x)[NCH]) const
    {
        if constexpr (!STAGE) {
#pragma unroll
            for (int u = 0; u < NCH; ++u) load(pos, e[u] & kIndexMask, x[u]);
        } else {
#pragma unroll
            for (int u = 0; u < NCH; ++u) get(min((unsigned)((e[u] & kIndexMask) - t0), (unsigned)kBlock - 1), x[u]);
#pragma unroll
            for (int u = 0; u < NCH; ++u)
                if ((unsigned)((e[u] & kIndexMask) - t0) >= (unsigned)kBlock) load(pos, e[u] & kIndexMask, x[u]);
        }
    }
};

// FP64 value tables in LDS as two planes of 16-byte halves {c0, c1}, {c2, c3}: at
// the 32-byte stride of the records a half could fall on half the banks only
// (density pass with staged records at 1,013,760 atoms: 65.2 -> 52.5 us).
template <typename R, int EV>
constexpr bool in_planes() { return EV == EV_TABLE && sizeof(R) == 8; }

template <typename R, int EV>
__device__ __forceinline__ void value_fill(R* dst, const R* src, int bins)
{
    if constexpr (in_planes<R, EV>()) {
        const double2* from = reinterpret_cast<const double2*>(src);
        double2* to = reinterpret_cast<double2*>(dst);
        for (int i = threadIdx.x; i < 2 * bins; i += blockDim.x) to[(i & 1) * bins + (i >> 1)] = from[i];
    } else {
        lds_fill(dst, src, bins * value_stride(EV));
    }
}

// density_term from the LDS copy of `bins` bins (LDS) or from global memory.
template <typename R, bool SINGLE, int NDK, int EV, bool LDS>
__device__ __forceinline__ R density_value(const PotArgs& P, const DevPotential& G, const R* tab, int si, int sj,
                                           double r)
{
    if constexpr (LDS && in_planes<R, EV>()) {
        const int bin = (int)(r * P.inv_w);
        const double u = fma(-(double)bin, P.w, r);
        const int at = (SINGLE ? 0 : si * G.ns + sj) * P.nbt + bin;
        const double2* t = reinterpret_cast<const double2*>(tab);
        const double2 lo = t[at], hi = t[(SINGLE ? 1 : P.ns * P.ns) * P.nbt + at];
        const double c[4] = {lo.x, lo.y, hi.x, hi.y};
        return cubic(c, u);
    } else {
        return density_term<R, SINGLE, NDK, EV>(P, G, tab, si, sj, r);
    }
}

// One neighbour's term of the density sum (Eq. Ucoh, the argument of F),
// accumulated in FP64 in both precision modes.
template <typename R, bool SINGLE, int NDK, int EV, int CMP, bool LDS>
__device__ __forceinline__ void density_pair(const PotArgs& P, const DevPotential& G, const R* tab,
                                             const DevReplica& Rp, const Box& bx, int e, int si, int sj,
                                             const double3& xi, const int4& qb, const double3& xj, const int4& qj,
                                             double& sum)
{
    const int code = ((unsigned)e >> kIndexBits) & kCodeMask;
    double dx, dy, dz;
    if (CMP) {
        compact_delta<CMP>(Rp, qb, qj, code, dx, dy, dz);
    } else {
        dx = xj.x - xi.x;
        dy = xj.y - xi.y;
        dz = xj.z - xi.z;
        if (code) apply_shift(bx, code, dx, dy, dz);
    }
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    if (!(r2 < P.rc2)) return;
    const double r = r2 * inv_dist<R>(r2);
    sum += (double)density_value<R, SINGLE, NDK, EV, LDS>(P, G, tab, si, sj, r);
}

// One neighbour's term of the force (and energy) sums.  tj: the neighbour's
// type byte (several species; one species reads it only for the virial of a
// rigid atom i, whose pairs with rigid atoms stay out of it).
template <typename R, bool SINGLE, int NPK, int NDK, int EV, int ENERGY, int CMP>
__device__ __forceinline__ void force_pair(const Buffers& b, int q, const PotArgs& P, const DevPotential& G,
                                           const R* tf, const R* te, const DevReplica& Rp, const Box& bx, int e,
                                           uint8_t ti, uint8_t tlist, const double4& pi, const int4& qb, R fpi,
                                           const double4& pj, const int4& qj, PairAcc& A)
{
    const int code = ((unsigned)e >> kIndexBits) & kCodeMask;
    double dx, dy, dz;
    R fpj;
    if (CMP) {
        compact_delta<CMP>(Rp, qb, qj, code, dx, dy, dz);
        fpj = (R)__int_as_float(qj.w);
    } else {
        dx = pj.x - pi.x;
        dy = pj.y - pi.y;
        dz = pj.z - pi.z;
        if (code) apply_shift(bx, code, dx, dy, dz);
        fpj = (R)pj.w;
    }
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    if (!(r2 < P.rc2)) return;
    const double ri = inv_dist<R>(r2);
    const double r = r2 * ri;
    const bool rigid_i = ti & kRigidBit;
    const uint8_t tj = !SINGLE ? tlist : (ENERGY == 1 && rigid_i) ? b.type[q][e & kIndexMask] : 0;
    R g, phi;
    pair_terms<R, SINGLE, NPK, NDK, EV, ENERGY>(P, G, tf, te, ti & 0x3F, tj & 0x3F, r, fpi, fpj, g, phi);
    accumulate<ENERGY>(A, (double)g * ri, dx, dy, dz, (double)phi, rigid_i && (tj & kRigidBit));
}

template <int ENERGY>
__device__ __forceinline__ void add_group(PairAcc& A, const PairAcc& G)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) A.f[a] += G.f[a];
    if (ENERGY == 1) A.epair += G.epair;
#pragma unroll
    for (int k = 0; k < (ENERGY == 1 || ENERGY == 3 ? 6 : ENERGY == 2 ? 3 : 0); ++k) A.w[k] += G.w[k];
}

__device__ __forceinline__ int4 list_group(const Buffers& b, int g, int64_t t, int64_t n_slots)
{
    return reinterpret_cast<const int4*>(b.nbr)[(int64_t)g * n_slots + t];
}
// neighbour type bytes of a group (several species)
template <bool SINGLE>
__device__ __forceinline__ uint32_t type_group(const Buffers& b, int g, int64_t t, int64_t n_slots)
{
    return SINGLE ? 0u : reinterpret_cast<const uint32_t*>(b.ntype)[(int64_t)g * n_slots + t];
}

// What the density pass leaves behind for one atom: F' for the force pass (in
// the compact records, in mixed precision) and F on energy steps.
template <bool SINGLE, int CMP>
__device__ __forceinline__ void density_epilogue(const Buffers& b, int p, int64_t t, const PotArgs& P,
                                                 const DevPotential& G, int si, const int4& qi, double rho, int energy)
{
    double F, dF;
    embed(SINGLE ? P.emb_c : G.emb_c[si], rho, F, dF);
    if (CMP) b.rec[1][t] = make_int4(qi.x, qi.y, qi.z, __float_as_int((float)dF));
    else reinterpret_cast<double*>(b.pos[p] + t)[3] = dF;
    if (energy) b.femb[t] = F;
}

// Density pass, one thread per atom.
template <typename R, bool SINGLE, int NPK, int NDK, int EV, int CMP, int NCH, bool TL, bool STAGE>
__global__ __launch_bounds__(TL ? kTableBlock : kBlock) void k_density(Buffers b, int p, int q, int64_t n_slots,
                                                                        PotArgs P, int energy)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t t0 = logical_block() * blockDim.x, t = t0 + threadIdx.x;
    const double4* __restrict__ pos = b.pos[p];
    const Stage<false> S(smem, (int)t0);
    // what the loop starts from is read before the tables, whose copy covers it
    double3 xi = make_double3(0.0, 0.0, 0.0);
    int4 qi = make_int4(0, 0, 0, 0);
    int rep = 0, si = 0, n = 0;
    if (t < n_slots) {
        rep = b.rep_of_wave[t / kWave];
        // the row's inner entries: the others lie beyond every density cutoff until the
        // next build (1,013,760 atoms, 17 of 28 entries: FP64 72 -> 59 us, mixed 56 -> 42)
        n = b.ninner[t];
        si = b.type[q][t] & 0x3F;
        if (CMP) qi = b.rec[0][t];
        else xi = load_xyz(pos, t);
        if (STAGE) S.put(threadIdx.x, xi);
    }
    const R* tab = tables<R>(b).dens;
    if (EV != EV_KNOTS && (SINGLE || TL)) {
        R* s = reinterpret_cast<R*>(smem + (STAGE ? S.kBytes : 0));
        value_fill<R, EV>(s, tab, (SINGLE ? 1 : P.ns * P.ns) * P.nbt);
        tab = s;
    }
    if (STAGE || (EV != EV_KNOTS && (SINGLE || TL))) __syncthreads();
    if (t >= n_slots) return;
    const DevReplica& Rp = b.reps[uniform(rep)];
    if (t - Rp.slot_off >= Rp.n_atoms) return;
    const Box bx = load_box(Rp);
    const DevPotential& G = *b.pot;
    const int4 qb = compact_base(qi);
    const __amdgpu_buffer_rsrc_t rs = record_rsrc(b.rec[0], n_slots);
    double rho = 0.0;
    constexpr int GR = NCH >= kChunk ? NCH / kChunk : 1;  // list groups per iteration
    constexpr int SUB = NCH >= kChunk ? 1 : kChunk / NCH;  // record batches per group
    static_assert(kChunk == 4 && NCH * SUB == kChunk * GR, "one int4 list load per four entries");
    constexpr bool AHEAD = CMP != 0;  // list groups read one round ahead (groups past cap are padding)
    int4 next[GR];
    uint32_t tnext[GR];
    if (AHEAD) {
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            next[g] = list_group(b, g, t, n_slots);
            tnext[g] = type_group<SINGLE>(b, g, t, n_slots);
        }
    }
    for (int k0 = 0; k0 < n; k0 += kChunk * GR) {
        int v[kChunk * GR];
        uint32_t tv[GR];
        double sum[GR];
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            if (!AHEAD) next[g] = list_group(b, (k0 >> 2) + g, t, n_slots);
            v[4 * g] = next[g].x;
            v[4 * g + 1] = next[g].y;
            v[4 * g + 2] = next[g].z;
            v[4 * g + 3] = next[g].w;
        }
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            tv[g] = AHEAD ? tnext[g] : type_group<SINGLE>(b, (k0 >> 2) + g, t, n_slots);
            sum[g] = 0.0;
        }
#pragma unroll
        for (int sb = 0; sb < SUB; ++sb) {
            const int kb = k0 + sb * NCH;
            if (kb >= n) break;
            int e[NCH];
            double3 xs[NCH];
            int4 qs[NCH];
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                e[u] = kb + u < n ? v[sb * NCH + u] : (int)t;
                if (CMP) qs[u] = record_load(rs, e[u] & kIndexMask);
            }
            if (!CMP) S.template gather<STAGE, NCH>(pos, e, xs);
            if (AHEAD && sb == 0 && k0 + kChunk * GR < n) {
#pragma unroll
                for (int g = 0; g < GR; ++g) {
                    next[g] = list_group(b, (k0 >> 2) + GR + g, t, n_slots);
                    tnext[g] = type_group<SINGLE>(b, (k0 >> 2) + GR + g, t, n_slots);
                }
            }
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                if (kb + u >= n) break;
                const int ku = sb * NCH + u;  // entry within the groups loaded
                const int sj = SINGLE ? 0 : (int)((tv[ku >> 2] >> (8 * (ku & 3))) & 0x3F);
                density_pair<R, SINGLE, NDK, EV, CMP, SINGLE || TL>(P, G, tab, Rp, bx, e[u], si, sj, xi, qb, xs[u], qs[u],
                                                      sum[ku >> 2]);
            }
        }
#pragma unroll
        for (int g = 0; g < GR; ++g) rho += sum[g];
    }
    density_epilogue<SINGLE, CMP>(b, p, t, P, G, si, qi, rho, energy);
}

// The split form: the groups of 64 atoms dealt to the kSplit waves of a
// workgroup (wave w takes groups w, w + kSplit, ...; lane l the l-th atom),
// whose sums wave 0 adds in order through LDS.
//
// What bounds a small system is the chain of dependent loads of one thread
// (list, records, list, ...: seven times ~2 us for 28 neighbours), on a chip it
// does not fill: at 2000 atoms 32 wavefronts for 1024 SIMDs.  Dealing the seven
// groups to eight waves leaves one link of that chain.  As the chip fills, the
// repeated prologues, table copies and exchanges of the sums through LDS cost
// more than that (KernelShape::split, split_sums).  Step times in us, one thread
// per atom against split in every pass, by slots (1.0 = 65,536, one one-thread
// wavefront per SIMD):
//   plain steps       one species FP64     mixed            two species FP64  mixed
//     1,984 (0.03)    34.7 -> 17.5     24.6 -> 15.9     50.0 -> 17.6     37.7 -> 16.4
//    64,896 (0.99)    37.5 -> 30.7     28.1 -> 24.5     53.1 -> 34.9     42.0 -> 26.4
//   100,352 (1.53)    42.2 -> 39.4     33.3 -> 32.3     56.4 -> 48.8     45.0 -> 36.2
//   126,720 (1.93)    45.9    45.7     35.8    36.2     59.1 -> 56.9     47.2 -> 41.5
//   168,704 (2.57)    52.0 <- 56.9     41.2 <- 44.0     60.3 <- 70.8     48.5 <- 50.6
//   energies every step
//    77,824 (1.19)    56.8 -> 55.0     48.7 -> 47.9     74.4 -> 61.0     63.8 -> 49.8
//    84,928 (1.30)    59.0    59.3     49.5 <- 50.9     74.5 -> 64.7     63.9 -> 52.0
//   108,672 (1.66)    59.0 <- 66.3     51.1 <- 56.3     76.1 -> 73.8     65.1 -> 58.0
//   126,720 (1.93)    62.8 <- 73.3     53.7 <- 62.2     78.6 <- 81.2     67.1 -> 64.1
//   168,704 (2.57)    70.7 <- 89.7     60.3 <- 75.3     79.9 <- 100      68.7 <- 76.3
// Barostat steps (virial) cross at 1.4 (FP64) and 1.3 with one species, 1.7 and 2.0
// with two; rows of 40 to 160 entries cross where those of 28 do.  The sums of a
// group are ten values instead of three: the force pass with sums goes back to one
// thread per atom earlier, the density pass beside it does not (126,720 atoms FP64
// with energies: force one thread, density either form 63 us).
//
// Four waves instead of eight: 22.1 us at 16,000 atoms (eight 18.7), 49.2 at
// 146,694 (51.6).


template <typename R, bool SINGLE, int NPK, int NDK, int EV, int CMP>
__global__ __launch_bounds__(kWave * kSplit) void k_density_split(Buffers b, int p, int q, int64_t n_slots, int cap,
                                                                  PotArgs P, int energy)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double part[kSplit - 1][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = uniform(threadIdx.x / kWave);
    const int64_t t = logical_block() * kWave + lane;  // one workgroup per wavefront of slots
    // the first group is read before anything that decides whether it is wanted
    int4 v4 = list_group(b, min(w, (cap - 1) >> 2), t, n_slots);
    uint32_t tv = type_group<SINGLE>(b, min(w, (cap - 1) >> 2), t, n_slots);
    const DevReplica& Rp = b.reps[uniform(b.rep_of_wave[t / kWave])];
    const bool pad = t - Rp.slot_off >= Rp.n_atoms;
    const Box bx = load_box(Rp);
    const DevPotential& G = *b.pot;
    const double4* __restrict__ pos = b.pos[p];
    const double3 xi = CMP ? make_double3(0.0, 0.0, 0.0) : load_xyz(pos, t);
    const int4 qi = CMP ? b.rec[0][t] : make_int4(0, 0, 0, 0);
    const int4 qb = compact_base(qi);
    const __amdgpu_buffer_rsrc_t rs = record_rsrc(b.rec[0], n_slots);
    const int si = b.type[q][t] & 0x3F;
    const int n = pad ? 0 : b.ninner[t];
    const R* tab = tables<R>(b).dens;
    if (EV != EV_KNOTS && SINGLE) {
        R* s = reinterpret_cast<R*>(smem);
        value_fill<R, EV>(s, tab, P.nbt);
        tab = s;
    }
    double rho = 0.0;
    for (int g0 = 0;; g0 += kSplit) {
        const int kb = (g0 + w) * kChunk;
        const int v[kChunk] = {v4.x, v4.y, v4.z, v4.w};
        int e[kChunk];
        double3 xs[kChunk];
        int4 qs[kChunk];
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            e[u] = kb + u < n ? v[u] : (int)t;
            if (kb + u < n) {
                if (CMP) qs[u] = record_load(rs, e[u] & kIndexMask);
                else xs[u] = load_xyz(pos, e[u] & kIndexMask);
            }
        }
        if (g0 == 0) __syncthreads();  // the tables
        double sum = 0.0;
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            if (kb + u >= n) break;
            const int sj = SINGLE ? 0 : (int)((tv >> (8 * u)) & 0x3F);
            density_pair<R, SINGLE, NDK, EV, CMP, SINGLE>(P, G, tab, Rp, bx, e[u], si, sj, xi, qb, xs[u], qs[u], sum);
        }
        const bool more = __ballot(n > (g0 + kSplit) * kChunk) != 0;  // alike in every wave
        if (more && kb + kSplit * kChunk < n) {
            v4 = list_group(b, g0 + kSplit + w, t, n_slots);
            tv = type_group<SINGLE>(b, g0 + kSplit + w, t, n_slots);
        }
        if (w) part[w - 1][lane] = sum;
        __syncthreads();
        if (w == 0) {
            rho += sum;
#pragma unroll
            for (int k = 0; k < kSplit - 1; ++k) rho += part[k][lane];
        }
        if (!more) break;
        __syncthreads();
    }
    if (w == 0 && !pad) density_epilogue<SINGLE, CMP>(b, p, t, P, G, si, qi, rho, energy);
}

// The force passes that close a thermostat or barostat step (closing kick, forces
// kept) also sum what its boundary needs per wavefront: the kinetic energy, or m v v
// and the virial.  (A pass of its own over velocities and virials before: 4.7 us per
// step, of 39 at 16,000 atoms under the barostat.)
template <int EN, bool CLOSE, bool OPEN, bool WRITEBACK>
constexpr bool boundary_sums()
{
    return CLOSE && !OPEN && !WRITEBACK && (EN == 0 || EN == 2 || EN == 3);
}

template <bool SINGLE, int EN>
__device__ __forceinline__ void wave_boundary_sums(const Buffers& b, int64_t t, const PotArgs& P, const DevPotential& G,
                                                   uint8_t ti, bool pad, const double (&v)[3], const PairAcc& A)
{
    constexpr int N = EN == 0 ? 1 : EN == 2 ? 6 : 12;
    double s[N] = {};
    if (!pad && !(ti & kRigidBit)) {
        const double hm = SINGLE ? P.half_m : G.half_m[ti & 0x3F], m = 2.0 * hm;
        if constexpr (EN == 0) {
            s[0] = hm * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
        } else if constexpr (EN == 2) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                s[a] = m * v[a] * v[a];
                s[3 + a] = A.w[a];
            }
        } else {
#pragma unroll
            for (int a = 0; a < 3; ++a) s[a] = m * v[a] * v[a];
            s[3] = m * v[0] * v[1];
            s[4] = m * v[0] * v[2];
            s[5] = m * v[1] * v[2];
#pragma unroll
            for (int k = 0; k < 6; ++k) s[6 + k] = A.w[k];
        }
    }
    double* out = EN == 0 ? b.nh_partial : b.pr_partial;
#pragma unroll
    for (int k = 0; k < N; ++k) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) s[k] += __shfl_xor(s[k], off, kWave);
        if ((threadIdx.x & (kWave - 1)) == 0) out[(t / kWave) * N + k] = s[k];
    }
}

// After the force sums of one atom: the integration and energy terms, the
// wavefront's energy sums (EN = 4) or boundary sums, and the compact record of the
// drifted position for the next density pass.  Called by all lanes of the
// wavefront where sums are taken.
template <bool SINGLE, int EN, bool CLOSE, bool OPEN, bool WRITEBACK, int CMP>
__device__ __forceinline__ void force_epilogue(const Buffers& b, int p, int q, int64_t t, int64_t n_slots,
                                               const DevReplica& Rp, const PotArgs& P, const DevPotential& G,
                                               double dt, const md_state& st, const double4& pi, uint8_t ti,
                                               const PairAcc& A, bool pad)
{
    constexpr bool WSUM = EN == 4, BSUM = boundary_sums<EN, CLOSE, OPEN, WRITEBACK>();
    double wv[kEnergyTerms] = {}, v[3] = {};
    if (!pad)
        atom_epilogue<SINGLE, WSUM ? 1 : EN, CLOSE, OPEN, WRITEBACK, WSUM || BSUM>(b, p, q, t, n_slots, Rp, P, G, dt, st,
                                                                                   pi, ti, A, wv, BSUM ? v : nullptr);
    if (WSUM) wave_sum_terms(b, t, wv);
    if constexpr (BSUM) wave_boundary_sums<SINGLE, EN>(b, t, P, G, ti, pad, v, A);
    if (CMP && OPEN && !pad) {
        const int4 c4 = b.cellxyz[t];
        const int c[3] = {c4.x, c4.y, c4.z};
        const double3 xn = load_xyz(b.pos[p ^ 1], t);
        int4 rq;
        if (!compact_coords<CMP>(Rp, c, xn.x, xn.y, xn.z, rq)) atomicAdd(&b.flags[F_COMPACT], 1);
        b.rec[0][t] = rq;
    }
}

// Wavefronts per SIMD the staged plain pass is held to.  (Not where it closes a
// thermostat step on tables with knots inside bins: held to six it spills, and a step
// of 1,013,760 atoms takes 252 us, 219 with the registers it asks for.)
template <int EV, int EN, bool CLOSE, bool OPEN, bool WRITEBACK, int NCH, bool STAGE>
constexpr int kForceWaves = STAGE && EN == 0 && NCH <= 4 &&
                                    !(EV == EV_SPLIT && boundary_sums<EN, CLOSE, OPEN, WRITEBACK>())
                                ? 6
                                : 1;

// Force pass + velocity Verlet, one thread per atom.
//
// EN = 4: the energies and virial of energy mode 1, summed per wavefront in the
// kernel (the reduction then reads one record per 64 atoms).
template <typename R, bool SINGLE, int NPK, int NDK, int EV, int EN, bool CLOSE, bool OPEN, bool WRITEBACK,
          int CMP, int NCH, bool TL, bool STAGE>
__global__ __launch_bounds__(TL ? kTableBlock : kBlock, (kForceWaves<EV, EN, CLOSE, OPEN, WRITEBACK, NCH, STAGE>)) void k_force(
    Buffers b, int p, int q, int64_t n_slots, PotArgs P, double dt, md_state st)
{
    constexpr bool WSUM = EN == 4;
    constexpr int ENERGY = WSUM ? 1 : EN;
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t t0 = logical_block() * blockDim.x, t = t0 + threadIdx.x;
    const double4* __restrict__ pos = b.pos[p];
    const Stage<true> S(smem, (int)t0);
    // what the loop starts from is read before the tables, whose copy covers it
    double4 pi = make_double4(0.0, 0.0, 0.0, 0.0);
    int4 qi = make_int4(0, 0, 0, 0);
    int rep = 0, n_row = 0;
    uint8_t ti = 0;
    if (t < n_slots) {
        rep = b.rep_of_wave[t / kWave];
        n_row = b.ncount[t];
        ti = b.type[q][t];
        if (CMP) qi = b.rec[1][t];
        else pi = pos[t];
        if (STAGE) S.put(threadIdx.x, pi);
    }
    const Tabs<R> T = tables<R>(b);
    const R* tf = T.force;
    const R* te = T.energy;
    if (EV != EV_KNOTS && (SINGLE || TL)) {
        const int nf = (SINGLE ? 1 : P.ns * P.ns) * P.nbt * force_stride(EV);
        R* s = reinterpret_cast<R*>(smem + (STAGE ? S.kBytes : 0));
        lds_fill(s, tf, nf);
        if (ENERGY == 1) lds_fill(s + nf, te, (SINGLE ? 1 : P.ns * P.ns) * P.nbt * value_stride(EV));
        tf = s;
        te = s + nf;
    }
    if (STAGE || (EV != EV_KNOTS && (SINGLE || TL))) __syncthreads();
    if (t >= n_slots) return;
    const DevReplica& Rp = b.reps[uniform(rep)];
    // slots past the replica's atoms leave, but for wavefront sums, which need every
    // lane (those lanes add zeros)
    const bool pad = t - Rp.slot_off >= Rp.n_atoms;
    if (pad && !WSUM && !boundary_sums<EN, CLOSE, OPEN, WRITEBACK>()) return;
    const Box bx = load_box(Rp);
    const DevPotential& G = *b.pot;
    const int4 qb = compact_base(qi);
    const __amdgpu_buffer_rsrc_t rs = record_rsrc(b.rec[1], n_slots);
    const int n = pad ? 0 : n_row;
    const R fpi = CMP ? (R)__int_as_float(qi.w) : (R)pi.w;
    PairAcc A;
    constexpr int GR = NCH >= kChunk ? NCH / kChunk : 1;  // list groups per iteration
    constexpr int SUB = NCH >= kChunk ? 1 : kChunk / NCH;  // record batches per group
    static_assert(kChunk == 4 && NCH * SUB == kChunk * GR, "one int4 list load per four entries");
    constexpr bool AHEAD = CMP != 0;  // list groups read one round ahead (groups past cap are padding)
    int4 next[GR];
    uint32_t tnext[GR];
    if (AHEAD) {
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            next[g] = list_group(b, g, t, n_slots);
            tnext[g] = type_group<SINGLE>(b, g, t, n_slots);
        }
    }
    for (int k0 = 0; k0 < n; k0 += kChunk * GR) {
        int v[kChunk * GR];
        uint32_t tv[GR];
        PairAcc sum[GR];
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            if (!AHEAD) next[g] = list_group(b, (k0 >> 2) + g, t, n_slots);
            v[4 * g] = next[g].x;
            v[4 * g + 1] = next[g].y;
            v[4 * g + 2] = next[g].z;
            v[4 * g + 3] = next[g].w;
        }
#pragma unroll
        for (int g = 0; g < GR; ++g) tv[g] = AHEAD ? tnext[g] : type_group<SINGLE>(b, (k0 >> 2) + g, t, n_slots);
#pragma unroll
        for (int sb = 0; sb < SUB; ++sb) {
            const int kb = k0 + sb * NCH;
            if (kb >= n) break;
            int e[NCH];
            double4 ps[NCH];
            int4 qs[NCH];
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                e[u] = kb + u < n ? v[sb * NCH + u] : (int)t;
                if (CMP) qs[u] = record_load(rs, e[u] & kIndexMask);
            }
            if (!CMP) S.template gather<STAGE, NCH>(pos, e, ps);
            if (AHEAD && sb == 0 && k0 + kChunk * GR < n) {
#pragma unroll
                for (int g = 0; g < GR; ++g) {
                    next[g] = list_group(b, (k0 >> 2) + GR + g, t, n_slots);
                    tnext[g] = type_group<SINGLE>(b, (k0 >> 2) + GR + g, t, n_slots);
                }
            }
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                if (kb + u >= n) break;
                const int ku = sb * NCH + u;  // entry within the groups loaded
                force_pair<R, SINGLE, NPK, NDK, EV, ENERGY, CMP>(b, q, P, G, tf, te, Rp, bx, e[u], ti,
                                                                 (uint8_t)(tv[ku >> 2] >> (8 * (ku & 3))), pi, qb, fpi,
                                                                 ps[u], qs[u], sum[ku >> 2]);
            }
        }
#pragma unroll
        for (int g = 0; g < GR; ++g) add_group<ENERGY>(A, sum[g]);
    }
    if (CMP) pi = pos[t];  // (the loop runs on the compact record)
    force_epilogue<SINGLE, EN, CLOSE, OPEN, WRITEBACK, CMP>(b, p, q, t, n_slots, Rp, P, G, dt, st, pi, ti, A, pad);
}

// Force pass + velocity Verlet, the groups of 64 atoms dealt to the kSplit waves
// of a workgroup; wave 0 adds the group sums in order and updates the atoms.
template <typename R, bool SINGLE, int NPK, int NDK, int EV, int EN, bool CLOSE, bool OPEN, bool WRITEBACK, int CMP>
__global__ __launch_bounds__(kWave * kSplit) void k_force_split(Buffers b, int p, int q, int64_t n_slots, int cap,
                                                                PotArgs P, double dt, md_state st)
{
    constexpr int ENERGY = EN == 4 ? 1 : EN;
    constexpr int NC = force_sums(EN);
    constexpr int W0 = ENERGY == 1 ? 4 : 3;  // first virial sum
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double part[kSplit - 1][NC][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = uniform(threadIdx.x / kWave);
    const int64_t t = logical_block() * kWave + lane;  // one workgroup per wavefront of slots
    // the first group is read before anything that decides whether it is wanted
    int4 v4 = list_group(b, min(w, (cap - 1) >> 2), t, n_slots);
    uint32_t tv = type_group<SINGLE>(b, min(w, (cap - 1) >> 2), t, n_slots);
    const DevReplica& Rp = b.reps[uniform(b.rep_of_wave[t / kWave])];
    const bool pad = t - Rp.slot_off >= Rp.n_atoms;
    const Box bx = load_box(Rp);
    const DevPotential& G = *b.pot;
    const double4* __restrict__ pos = b.pos[p];
    const double4 pi = pos[t];
    const int4 qi = CMP ? b.rec[1][t] : make_int4(0, 0, 0, 0);
    const int4 qb = compact_base(qi);
    const __amdgpu_buffer_rsrc_t rs = record_rsrc(b.rec[1], n_slots);
    const uint8_t ti = b.type[q][t];
    const int n = pad ? 0 : b.ncount[t];
    const R fpi = CMP ? (R)__int_as_float(qi.w) : (R)pi.w;
    const R* tf = tables<R>(b).force;
    const R* te = tables<R>(b).energy;
    if (EV != EV_KNOTS && SINGLE) {
        const int nf = P.nbt * force_stride(EV);
        R* s = reinterpret_cast<R*>(smem);
        lds_fill(s, tf, nf);
        if (ENERGY == 1) lds_fill(s + nf, te, P.nbt * value_stride(EV));
        tf = s;
        te = s + nf;
    }
    PairAcc A;
    for (int g0 = 0;; g0 += kSplit) {
        const int kb = (g0 + w) * kChunk;
        const int v[kChunk] = {v4.x, v4.y, v4.z, v4.w};
        int e[kChunk];
        double4 ps[kChunk];
        int4 qs[kChunk];
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            e[u] = kb + u < n ? v[u] : (int)t;
            if (kb + u < n) {
                if (CMP) qs[u] = record_load(rs, e[u] & kIndexMask);
                else ps[u] = pos[e[u] & kIndexMask];
            }
        }
        if (g0 == 0) __syncthreads();  // the tables
        PairAcc sum;
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            if (kb + u >= n) break;
            force_pair<R, SINGLE, NPK, NDK, EV, ENERGY, CMP>(b, q, P, G, tf, te, Rp, bx, e[u], ti,
                                                             (uint8_t)(tv >> (8 * u)), pi, qb, fpi, ps[u], qs[u], sum);
        }
        const bool more = __ballot(n > (g0 + kSplit) * kChunk) != 0;  // alike in every wave
        if (more && kb + kSplit * kChunk < n) {
            v4 = list_group(b, g0 + kSplit + w, t, n_slots);
            tv = type_group<SINGLE>(b, g0 + kSplit + w, t, n_slots);
        }
        if (w) {
            double(*mine)[kWave] = part[w - 1];
#pragma unroll
            for (int a = 0; a < 3; ++a) mine[a][lane] = sum.f[a];
            if (ENERGY == 1) mine[3][lane] = sum.epair;
#pragma unroll
            for (int k = 0; k < NC - W0; ++k) mine[W0 + k][lane] = sum.w[k];
        }
        __syncthreads();
        if (w == 0) {
            add_group<ENERGY>(A, sum);
#pragma unroll
            for (int j = 0; j < kSplit - 1; ++j) {
                PairAcc o;
#pragma unroll
                for (int a = 0; a < 3; ++a) o.f[a] = part[j][a][lane];
                if (ENERGY == 1) o.epair = part[j][3][lane];
#pragma unroll
                for (int k = 0; k < NC - W0; ++k) o.w[k] = part[j][W0 + k][lane];
                add_group<ENERGY>(A, o);
            }
        }
        if (!more) break;
        __syncthreads();
    }
    if (w == 0) force_epilogue<SINGLE, EN, CLOSE, OPEN, WRITEBACK, CMP>(b, p, q, t, n_slots, Rp, P, G, dt, st, pi, ti, A, pad);
}

// ---------------------------------------------------------------------------
// Half-list variant (MD_NBR_HALF_ATOMIC): the comparison form in which every
// unordered pair is evaluated once, by its lower slot, and the partner's share
// goes to memory with FP64 atomics; the paper's own OpenMP code resolves the
// same write conflict with link-cell locks (section "OpenMP Parallelisation").
// Density: rho_i and rho_j both receive their term; the embedding then runs as
// its own pass.  Forces: f_i += s d, f_j -= s d; pair energies split in halves;
// the virial counts every pair once.  Integration follows as a separate pass.

// Density pass, half list: accumulates into rhalf (zeroed beforehand).
template <typename R, bool SINGLE, int NPK, int NDK, int EV>
__global__ __launch_bounds__(kBlock) void k_density_half(Buffers b, int p, int q, int64_t n_slots, PotArgs P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const R* tab = tables<R>(b).dens;
    if (EV != EV_KNOTS && SINGLE) {
        R* s = reinterpret_cast<R*>(smem);
        lds_fill(s, tab, P.nbt * value_stride(EV));
        __syncthreads();
        tab = s;
    }
    const int64_t t = global_thread();
    if (t >= n_slots) return;
    const DevReplica& Rp = b.reps[uniform(b.rep_of_wave[t / kWave])];
    if (t - Rp.slot_off >= Rp.n_atoms) return;
    const Box bx = load_box(Rp);
    const DevPotential& G = *b.pot;
    const double4* __restrict__ pos = b.pos[p];
    const int32_t* __restrict__ nbr = b.nbr;
    const double3 xi = load_xyz(pos, t);
    const int si = b.type[q][t] & 0x3F;
    const int n = b.ncount[t];
    double rho = 0.0;
    for (int k = 0; k < n; ++k) {
        const int e = nbr[nbr_at(k, t, n_slots)];
        const int j = e & kIndexMask;
        const double3 xj = load_xyz(pos, j);
        double dx = xj.x - xi.x, dy = xj.y - xi.y, dz = xj.z - xi.z;
        const int code = ((unsigned)e >> kIndexBits) & kCodeMask;
        if (code) apply_shift(bx, code, dx, dy, dz);
        const double r2 = dx * dx + dy * dy + dz * dz;
        if (!(r2 < P.rc2)) continue;
        const double r = r2 * inv_dist<R>(r2);
        const int sj = SINGLE ? 0 : (b.type[q][j] & 0x3F);
        const R to_i = density_term<R, SINGLE, NDK, EV>(P, G, tab, si, sj, r);
        const R to_j = SINGLE ? to_i : density_term<R, SINGLE, NDK, EV>(P, G, tab, sj, si, r);
        rho += (double)to_i;
        atomicAdd(&b.rhalf[j], (double)to_j);
    }
    atomicAdd(&b.rhalf[t], rho);
}

// Embedding after the half-list density pass: F_i, F'_i from rho_i.
template <bool SINGLE>
__global__ void k_embed_half(Buffers b, int p, int q, int64_t n_slots, PotArgs P, int energy)
{
    const int64_t t = global_thread();
    if (t >= n_slots) return;
    const DevReplica& Rp = b.reps[uniform(b.rep_of_wave[t / kWave])];
    if (t - Rp.slot_off >= Rp.n_atoms) return;
    const DevPotential& G = *b.pot;
    const int si = b.type[q][t] & 0x3F;
    double F, dF;
    embed(SINGLE ? P.emb_c : G.emb_c[si], b.rhalf[t], F, dF);
    reinterpret_cast<double*>(b.pos[p] + t)[3] = dF;
    if (energy) b.femb[t] = F;
}

// Force pass, half list: forces and pair energies into fhalf / ehalf (zeroed
// beforehand); the virial of the pairs an atom owns into its energy slots.
template <typename R, bool SINGLE, int NPK, int NDK, int EV, bool ENERGY>
__global__ __launch_bounds__(kBlock) void k_force_half(Buffers b, int p, int q, int64_t n_slots, PotArgs P)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const Tabs<R> T = tables<R>(b);
    const R* tf = T.force;
    const R* te = T.energy;
    if (EV != EV_KNOTS && SINGLE) {
        R* s = reinterpret_cast<R*>(smem);
        lds_fill(s, tf, P.nbt * force_stride(EV));
        if (ENERGY == 1) lds_fill(s + P.nbt * force_stride(EV), te, P.nbt * value_stride(EV));
        __syncthreads();
        tf = s;
        te = s + P.nbt * force_stride(EV);
    }
    const int64_t t = global_thread();
    if (t >= n_slots) return;
    const DevReplica& Rp = b.reps[uniform(b.rep_of_wave[t / kWave])];
    if (t - Rp.slot_off >= Rp.n_atoms) return;
    const Box bx = load_box(Rp);
    const DevPotential& G = *b.pot;
    const double4* __restrict__ pos = b.pos[p];
    const int32_t* __restrict__ nbr = b.nbr;
    const double4 pi = pos[t];
    const uint8_t ti = b.type[q][t];
    const int si = ti & 0x3F;
    const bool rigid_i = ti & kRigidBit;
    const int n = b.ncount[t];
    PairAcc A;
    for (int k = 0; k < n; ++k) {
        const int e = nbr[nbr_at(k, t, n_slots)];
        const int j = e & kIndexMask;
        const double4 pj = pos[j];
        double dx = pj.x - pi.x, dy = pj.y - pi.y, dz = pj.z - pi.z;
        const int code = ((unsigned)e >> kIndexBits) & kCodeMask;
        if (code) apply_shift(bx, code, dx, dy, dz);
        const double r2 = dx * dx + dy * dy + dz * dz;
        if (!(r2 < P.rc2)) continue;
        const double ri = inv_dist<R>(r2);
        const double r = r2 * ri;
        const uint8_t tj = (!SINGLE || ENERGY) ? b.type[q][j] : 0;
        R g, phi;
        pair_terms<R, SINGLE, NPK, NDK, EV, ENERGY>(P, G, tf, te, si, tj & 0x3F, r, (R)pi.w, (R)pj.w, g, phi);
        const double s = (double)g * ri;
        accumulate<ENERGY>(A, s, dx, dy, dz, (double)phi, rigid_i && (tj & kRigidBit));
        atomicAdd(&b.fhalf[0][j], -s * dx);
        atomicAdd(&b.fhalf[1][j], -s * dy);
        atomicAdd(&b.fhalf[2][j], -s * dz);
        if (ENERGY) atomicAdd(&b.ehalf[j], 0.5 * (double)phi);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) atomicAdd(&b.fhalf[a][t], A.f[a]);
    if (ENERGY) {
        atomicAdd(&b.ehalf[t], 0.5 * A.epair);
#pragma unroll
        for (int k = 0; k < 6; ++k) b.eslot[(int64_t)(E_W0 + k) * n_slots + t] = A.w[k];
    }
}

// Velocity Verlet and energy terms after the half-list force pass.
template <bool SINGLE, bool ENERGY, bool CLOSE, bool OPEN, bool WRITEBACK>
__global__ void k_integrate_half(Buffers b, int p, int q, int64_t n_slots, PotArgs P, double dt, md_state st)
{
    const int64_t t = global_thread();
    if (t >= n_slots) return;
    const DevReplica& Rp = b.reps[uniform(b.rep_of_wave[t / kWave])];
    if (t - Rp.slot_off >= Rp.n_atoms) return;
    const DevPotential& G = *b.pot;
    PairAcc A;
#pragma unroll
    for (int a = 0; a < 3; ++a) A.f[a] = b.fhalf[a][t];
    if (ENERGY) {
        A.epair = 2.0 * b.ehalf[t];
#pragma unroll
        for (int k = 0; k < 6; ++k) A.w[k] = b.eslot[(int64_t)(E_W0 + k) * n_slots + t];
    }
    atom_epilogue<SINGLE, ENERGY, CLOSE, OPEN, WRITEBACK>(b, p, q, t, n_slots, Rp, P, G, dt, st, b.pos[p][t],
                                                         b.type[q][t], A);
}

}  // namespace

template <typename R, bool S, int NP, int ND, int EV, int CMP, bool TL, bool STAGE>
static void density_chunked(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int energy,
                            size_t lds, hipStream_t s)
{
    const int block = TL ? kTableBlock : kBlock;
    const dim3 grid((unsigned)((k.n_slots + block - 1) / block));
    if (k.nchunk == 2)
        hipLaunchKernelGGL((k_density<R, S, NP, ND, EV, CMP, 2, TL, STAGE>), grid, dim3(block), lds, s, b, p, q,
                           k.n_slots, P, energy);
    else if (k.nchunk == 8)
        hipLaunchKernelGGL((k_density<R, S, NP, ND, EV, CMP, 8, TL, STAGE>), grid, dim3(block), lds, s, b, p, q,
                           k.n_slots, P, energy);
    else
        hipLaunchKernelGGL((k_density<R, S, NP, ND, EV, CMP, 4, TL, STAGE>), grid, dim3(block), lds, s, b, p, q,
                           k.n_slots, P, energy);
}

template <typename R, bool S, int NP, int ND, int EV, int CMP>
static void density_tables(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int energy,
                           hipStream_t s)
{
    const size_t split_lds = S && EV != EV_KNOTS ? (size_t)P.nbt * value_stride(EV) * sizeof(R) : 0;
    if (k.split && split_fits(split_lds, 1)) {
        hipLaunchKernelGGL((k_density_split<R, S, NP, ND, EV, CMP>), dim3((unsigned)(k.n_slots / kWave)),
                           dim3(kWave * kSplit), split_lds, s, b, p, q, k.n_slots, k.cap, P, energy);
        return;
    }
    // tables in LDS: always for one species, for several when they fit
    const size_t bytes = EV != EV_KNOTS ? (size_t)(S ? 1 : P.ns * P.ns) * P.nbt * value_stride(EV) * sizeof(R) : 0;
    if constexpr (!S && EV != EV_KNOTS) {
        if (bytes <= (size_t)k.lds_limit) {
            density_chunked<R, S, NP, ND, EV, CMP, true, false>(b, p, q, k, P, energy, bytes, s);
            return;
        }
    }
    if constexpr (S && sizeof(R) == 8) {
        if (k.stage && bytes + Stage<false>::kBytes <= kStageLds<false>) {
            density_chunked<R, S, NP, ND, EV, CMP, false, true>(b, p, q, k, P, energy, bytes + Stage<false>::kBytes, s);
            return;
        }
    }
    density_chunked<R, S, NP, ND, EV, CMP, false, false>(b, p, q, k, P, energy, S ? bytes : 0, s);
}

template <typename R, bool S, int NP, int ND, int EV>
static void density_variant(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int energy,
                            hipStream_t s)
{
    if constexpr (sizeof(R) == 4) {  // compact records: mixed precision only
        if (k.compact == 2) return density_tables<R, S, NP, ND, EV, 2>(b, p, q, k, P, energy, s);
        if (k.compact) return density_tables<R, S, NP, ND, EV, 1>(b, p, q, k, P, energy, s);
    }
    density_tables<R, S, NP, ND, EV, 0>(b, p, q, k, P, energy, s);
}

template <typename R, bool S, int NP, int ND, int EV>
static void density_half_variant(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int energy,
                                 hipStream_t s)
{
    const size_t lds = (EV != EV_KNOTS && S) ? (size_t)P.nbt * value_stride(EV) * sizeof(R) : 0;
    const dim3 grid(blocks_for(k.n_slots));
    launch_fill_f64(b.rhalf, 0.0, k.n_slots, s);
    hipLaunchKernelGGL((k_density_half<R, S, NP, ND, EV>), grid, dim3(kBlock), lds, s, b, p, q, k.n_slots, P);
    hipLaunchKernelGGL((k_embed_half<S>), grid, dim3(kBlock), 0, s, b, p, q, k.n_slots, P, energy);
}

template <typename R, bool S>
static void density_dispatch(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int half_list,
                             int energy, hipStream_t s)
{
    // the term-by-term knot sums are FP64 only (the runtime refuses them in mixed precision)
    constexpr bool knots = sizeof(R) == 8;
    if (half_list) {
        if (k.table == 2) density_half_variant<R, S, 8, 8, EV_SPLIT>(b, p, q, k, P, energy, s);
        else if (k.table || !knots) density_half_variant<R, S, 8, 8, EV_TABLE>(b, p, q, k, P, energy, s);
        else if constexpr (knots) {
            if (k.ndk == 2) density_half_variant<R, S, 6, 2, EV_KNOTS>(b, p, q, k, P, energy, s);  // density knots only
            else density_half_variant<R, S, 8, 8, EV_KNOTS>(b, p, q, k, P, energy, s);
        }
        return;
    }
    if (k.table == 2) density_variant<R, S, 8, 8, EV_SPLIT>(b, p, q, k, P, energy, s);
    else if (k.table || !knots) density_variant<R, S, 8, 8, EV_TABLE>(b, p, q, k, P, energy, s);
    else if constexpr (knots) {
        if (k.ndk == 2) density_variant<R, S, 6, 2, EV_KNOTS>(b, p, q, k, P, energy, s);  // density knots only
        else density_variant<R, S, 8, 8, EV_KNOTS>(b, p, q, k, P, energy, s);
    }
}
// The neighbour chunk applies to the velocity-Verlet step kernels (with and
// without energies) and to the plain force pass the autotuner times; the other
// variants run once per call or per barostat step.
template <typename R, bool S, int NP, int ND, int EV, int E, bool C, bool O, bool W, int CMP, bool TL, bool STAGE>
static void force_chunked(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, double dt_fs,
                          const md_state& st, size_t lds, hipStream_t s)
{
    const int block = TL ? kTableBlock : kBlock;
    const dim3 grid((unsigned)((k.n_slots + block - 1) / block));
    constexpr bool step = ((E == 0 || E == 4) && C && O && !W) || (E == 0 && !C && !O && !W);
    if constexpr (step) {
        if (k.nchunk == 2) {
            hipLaunchKernelGGL((k_force<R, S, NP, ND, EV, E, C, O, W, CMP, 2, TL, STAGE>), grid, dim3(block), lds, s, b,
                               p, q, k.n_slots, P, dt_fs, st);
            return;
        }
        if (k.nchunk == 8) {
            hipLaunchKernelGGL((k_force<R, S, NP, ND, EV, E, C, O, W, CMP, 8, TL, STAGE>), grid, dim3(block), lds, s, b,
                               p, q, k.n_slots, P, dt_fs, st);
            return;
        }
    }
    hipLaunchKernelGGL((k_force<R, S, NP, ND, EV, E, C, O, W, CMP, 4, TL, STAGE>), grid, dim3(block), lds, s, b, p, q,
                       k.n_slots, P, dt_fs, st);
}

template <typename R, bool S, int NP, int ND, int EV, int E, bool C, bool O, bool W, int CMP>
static void force_tables(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, double dt_fs,
                         const md_state& st, hipStream_t s)
{
    const size_t split_lds =
        S && EV != EV_KNOTS ? (size_t)P.nbt * (force_stride(EV) + (E == 1 || E == 4 ? value_stride(EV) : 0)) * sizeof(R)
                            : 0;
    if ((E == 0 ? k.split : k.split_sums) && split_fits(split_lds, force_sums(E))) {
        hipLaunchKernelGGL((k_force_split<R, S, NP, ND, EV, E, C, O, W, CMP>), dim3((unsigned)(k.n_slots / kWave)),
                           dim3(kWave * kSplit), split_lds, s, b, p, q, k.n_slots, k.cap, P, dt_fs, st);
        return;
    }
    // tables in LDS: always for one species, for several when they fit
    const size_t bytes = EV != EV_KNOTS ? (size_t)(S ? 1 : P.ns * P.ns) * P.nbt *
                                              (force_stride(EV) + (E == 1 || E == 4 ? value_stride(EV) : 0)) *
                                              sizeof(R)
                                        : 0;
    if constexpr (!S && EV != EV_KNOTS) {
        if (bytes <= (size_t)k.lds_limit) {
            force_chunked<R, S, NP, ND, EV, E, C, O, W, CMP, true, false>(b, p, q, k, P, dt_fs, st, bytes, s);
            return;
        }
    }
    if constexpr (S && sizeof(R) == 8) {
        if (k.stage && bytes + Stage<true>::kBytes <= kStageLds<true>) {
            force_chunked<R, S, NP, ND, EV, E, C, O, W, CMP, false, true>(b, p, q, k, P, dt_fs, st,
                                                                         bytes + Stage<true>::kBytes, s);
            return;
        }
    }
    force_chunked<R, S, NP, ND, EV, E, C, O, W, CMP, false, false>(b, p, q, k, P, dt_fs, st, S ? bytes : 0, s);
}

template <typename R, bool S, int NP, int ND, int EV, int E, bool C, bool O, bool W>
static void force_launch(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, double dt_fs,
                         const md_state& st, hipStream_t s)
{
    if constexpr (sizeof(R) == 4) {  // compact records: mixed precision only
        if (k.compact == 2) return force_tables<R, S, NP, ND, EV, E, C, O, W, 2>(b, p, q, k, P, dt_fs, st, s);
        if (k.compact) return force_tables<R, S, NP, ND, EV, E, C, O, W, 1>(b, p, q, k, P, dt_fs, st, s);
    }
    force_tables<R, S, NP, ND, EV, E, C, O, W, 0>(b, p, q, k, P, dt_fs, st, s);
}

template <typename R, bool S, int NP, int ND, int EV>
static void force_variant(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, ForceFlags fl,
                          double dt_fs, const md_state& st, hipStream_t s)
{
    if (!fl.close && !fl.open) {
        if (!fl.writeback && fl.energy == 3)  // full-matrix barostat: the whole virial tensor, forces kept
            force_launch<R, S, NP, ND, EV, 3, false, false, false>(b, p, q, k, P, dt_fs, st, s);
        else if (!fl.writeback && fl.energy)  // barostat: the stress of the starting state, forces kept
            force_launch<R, S, NP, ND, EV, 2, false, false, false>(b, p, q, k, P, dt_fs, st, s);
        else if (!fl.writeback) force_launch<R, S, NP, ND, EV, false, false, false, false>(b, p, q, k, P, dt_fs, st, s);
        else if (fl.energy == 4) force_launch<R, S, NP, ND, EV, 4, false, false, true>(b, p, q, k, P, dt_fs, st, s);
        else if (fl.energy) force_launch<R, S, NP, ND, EV, true, false, false, true>(b, p, q, k, P, dt_fs, st, s);
        else force_launch<R, S, NP, ND, EV, false, false, false, true>(b, p, q, k, P, dt_fs, st, s);
    } else if (!fl.close && fl.open) {
        force_launch<R, S, NP, ND, EV, false, false, true, false>(b, p, q, k, P, dt_fs, st, s);
    } else if (fl.close && fl.open) {
        if (fl.energy)  // per-step energies, summed per wavefront (mode 4; no other comes here)
            force_launch<R, S, NP, ND, EV, 4, true, true, false>(b, p, q, k, P, dt_fs, st, s);
        else force_launch<R, S, NP, ND, EV, false, true, true, false>(b, p, q, k, P, dt_fs, st, s);
    } else if (!fl.writeback && fl.energy == 3) {  // full-matrix barostat: closing kick, virial tensor
        force_launch<R, S, NP, ND, EV, 3, true, false, false>(b, p, q, k, P, dt_fs, st, s);
    } else if (!fl.writeback && fl.energy) {  // barostat: closing kick with the stress, forces kept
        force_launch<R, S, NP, ND, EV, 2, true, false, false>(b, p, q, k, P, dt_fs, st, s);
    } else if (!fl.writeback) {
        force_launch<R, S, NP, ND, EV, false, true, false, false>(b, p, q, k, P, dt_fs, st, s);
    } else if (fl.energy == 4) {  // the last step of a velocity-Verlet call
        force_launch<R, S, NP, ND, EV, 4, true, false, true>(b, p, q, k, P, dt_fs, st, s);
    } else {
        force_launch<R, S, NP, ND, EV, true, true, false, true>(b, p, q, k, P, dt_fs, st, s);
    }
}

template <bool S, bool E, bool C, bool O, bool W>
static void integrate_half(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, double dt_fs,
                           const md_state& st, hipStream_t s)
{
    hipLaunchKernelGGL((k_integrate_half<S, E, C, O, W>), dim3(blocks_for(k.n_slots)), dim3(kBlock), 0, s, b, p, q,
                       k.n_slots, P, dt_fs, st);
}

template <typename R, bool S, int NP, int ND, int EV>
static void force_half_variant(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, ForceFlags fl,
                               double dt_fs, const md_state& st, hipStream_t s)
{
    const dim3 grid(blocks_for(k.n_slots));
    for (int a = 0; a < 3; ++a) launch_fill_f64(b.fhalf[a], 0.0, k.n_slots, s);
    if (fl.energy) launch_fill_f64(b.ehalf, 0.0, k.n_slots, s);
    const size_t lds =
        (EV != EV_KNOTS && S) ? (size_t)P.nbt * (force_stride(EV) + (fl.energy ? value_stride(EV) : 0)) * sizeof(R) : 0;
    if (fl.energy)
        hipLaunchKernelGGL((k_force_half<R, S, NP, ND, EV, true>), grid, dim3(kBlock), lds, s, b, p, q, k.n_slots, P);
    else
        hipLaunchKernelGGL((k_force_half<R, S, NP, ND, EV, false>), grid, dim3(kBlock), lds, s, b, p, q, k.n_slots, P);
    if (!fl.close && !fl.open) {
        if (!fl.writeback) integrate_half<S, false, false, false, false>(b, p, q, k, P, dt_fs, st, s);
        else if (fl.energy) integrate_half<S, true, false, false, true>(b, p, q, k, P, dt_fs, st, s);
        else integrate_half<S, false, false, false, true>(b, p, q, k, P, dt_fs, st, s);
    } else if (!fl.close && fl.open) {
        integrate_half<S, false, false, true, false>(b, p, q, k, P, dt_fs, st, s);
    } else if (fl.close && fl.open) {
        if (fl.energy) integrate_half<S, true, true, true, false>(b, p, q, k, P, dt_fs, st, s);
        else integrate_half<S, false, true, true, false>(b, p, q, k, P, dt_fs, st, s);
    } else if (!fl.writeback) {
        integrate_half<S, false, true, false, false>(b, p, q, k, P, dt_fs, st, s);
    } else {
        integrate_half<S, true, true, false, true>(b, p, q, k, P, dt_fs, st, s);
    }
}

template <typename R, bool S>
static void force_dispatch(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int half_list,
                           ForceFlags fl, double dt_fs, const md_state& st, hipStream_t s)
{
    constexpr bool knots = sizeof(R) == 8;  // knot sums: FP64 only
    if (half_list) {
        if (k.table == 2) force_half_variant<R, S, 8, 8, EV_SPLIT>(b, p, q, k, P, fl, dt_fs, st, s);
        else if (k.table || !knots) force_half_variant<R, S, 8, 8, EV_TABLE>(b, p, q, k, P, fl, dt_fs, st, s);
        else if constexpr (knots) {
            if (k.npk == 6 && k.ndk == 2) force_half_variant<R, S, 6, 2, EV_KNOTS>(b, p, q, k, P, fl, dt_fs, st, s);
            else if (k.npk <= 8 && k.ndk <= 8) force_half_variant<R, S, 8, 8, EV_KNOTS>(b, p, q, k, P, fl, dt_fs, st, s);
            else if constexpr (S) force_half_variant<R, S, 16, 4, EV_KNOTS>(b, p, q, k, P, fl, dt_fs, st, s);
        }
        return;
    }
    if (k.table == 2) force_variant<R, S, 8, 8, EV_SPLIT>(b, p, q, k, P, fl, dt_fs, st, s);
    else if (k.table || !knots) force_variant<R, S, 8, 8, EV_TABLE>(b, p, q, k, P, fl, dt_fs, st, s);
    else if constexpr (knots) {
        if (k.npk == 6 && k.ndk == 2) force_variant<R, S, 6, 2, EV_KNOTS>(b, p, q, k, P, fl, dt_fs, st, s);
        else if (k.npk <= 8 && k.ndk <= 8) force_variant<R, S, 8, 8, EV_KNOTS>(b, p, q, k, P, fl, dt_fs, st, s);
        else if constexpr (S) force_variant<R, S, 16, 4, EV_KNOTS>(b, p, q, k, P, fl, dt_fs, st, s);
    }
}
// Instantiated by one translation unit each.
template <typename R, bool S>
void density_of(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int half_list, int energy,
                hipStream_t s)
{
    density_dispatch<R, S>(b, p, q, k, P, half_list, energy, s);
}
template <typename R, bool S>
void force_of(const Buffers& b, int p, int q, const KernelShape& k, const PotArgs& P, int half_list, ForceFlags fl,
              double dt_fs, const md_state& st, hipStream_t s)
{
    force_dispatch<R, S>(b, p, q, k, P, half_list, fl, dt_fs, st, s);
}

}  // namespace mdk
