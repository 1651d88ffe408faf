// gfx950 kernels of the list build (paper, "The Neighbourlist calculation"):
// binning of the atoms into link cells, the scan of the cell populations, the
// counting sort into cell order (atoms within a cell ordered by caller index),
// the gather of the atom state into the new slot order, the cell adjacency
// table and the Verlet list itself; and the automatic rebuild's displacement
// check with the gating every build kernel takes.
#include "md_device.h"

namespace mdk {
namespace {
// counter[key] += 1 for every lane with key >= 0; returns the lane's old value
// plus its rank among the lanes of its run.  Lanes with equal keys usually sit
// side by side (the slots are cell-sorted from the previous build), so each
// run of equal keys issues one atomic instead of one per lane.  Must be called
// by every lane of the wavefront.
__device__ __forceinline__ int wave_run_add(int32_t* counter, int key)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int prev = __shfl_up(key, 1, kWave);
    const uint64_t heads = __ballot(lane == 0 || key != prev);
    const uint64_t upto = lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1);
    const int head = 63 - __clzll(heads & upto);  // first lane of this run
    const uint64_t later = heads & ~upto;
    const int next = later ? __ffsll((unsigned long long)later) - 1 : kWave;
    int base = 0;
    if (lane == head && key >= 0) base = atomicAdd(&counter[key], next - lane);
    base = __shfl(base, head, kWave);
    return base + (lane - head);
}


// ---------------------------------------------------------------------------
// Rebuild stage 1 of 4: link cell of every atom, cell populations, and the skin
// guard (net displacement since the previous build must stay below skin/2).
// Every rebuild kernel takes `gate`: NULL for a build of all replicas, else
// the automatic rebuild's flags, and then it leaves alone every replica r with
// gate[1 + r] == 0 (slot ranges and link cells are per replica, so a kept
// replica's slots, cells and list stay exactly as they are).  Gated builds run
// at every step and mostly find nothing flagged: they launch a capped grid
// whose threads stride over the elements (whole wavefronts per stride, as
// replicas are wave aligned), so that such a launch ends at once; builds of
// all replicas take one element per thread.
constexpr int64_t kGatedBlocks = 2048;

__device__ __forceinline__ bool replica_kept(const Buffers& b, const int32_t* gate, int64_t t)
{
    return gate && gate[1 + uniform(b.rep_of_wave[t / kWave])] == 0;
}

__device__ __forceinline__ void bin_slot(const Buffers& b, int p, int q, int64_t t, double half_skin2, int check_skin)
{
    const DevReplica& R = b.reps[uniform(b.rep_of_wave[t / kWave])];
    const bool valid = b.id[q][t] >= 0;
    const Box bx = load_box(R);
    const double3 x = load_xyz(b.pos[p], t);
    int c[3];
    cell_coords(bx, x.x, x.y, x.z, c);
    const int cell = valid ? cell_index(R, c[0], c[1], c[2]) : -1;
    b.cell_of[t] = cell;
    wave_run_add(b.bin_count, cell);
    if (!valid) return;
    if (check_skin) {
        // displacement since the build, after mapping the build position into
        // the current box (the two boxes differ only under the barostat)
        const double3 x0 = load_xyz(b.xbuild, t);
        double dx, dy, dz;
        if (bx.tri) {  // strained by the homogeneous map mb since the build
            const double u[3] = {x0.x - bx.o[0], x0.y - bx.o[1], x0.z - bx.o[2]};
            dx = (x.x - bx.o[0]) - (R.mb[0] * u[0] + R.mb[1] * u[1] + R.mb[2] * u[2]);
            dy = (x.y - bx.o[1]) - (R.mb[3] * u[0] + R.mb[4] * u[1] + R.mb[5] * u[2]);
            dz = (x.z - bx.o[2]) - (R.mb[6] * u[0] + R.mb[7] * u[1] + R.mb[8] * u[2]);
        } else {
            dx = (x.x - bx.o[0]) - (x0.x - bx.o[0]) * (R.box[0] / R.lbuild[0]);
            dy = (x.y - bx.o[1]) - (x0.y - bx.o[1]) * (R.box[1] / R.lbuild[1]);
            dz = (x.z - bx.o[2]) - (x0.z - bx.o[2]) * (R.box[2] / R.lbuild[2]);
        }
        if (dx * dx + dy * dy + dz * dz > half_skin2) atomicAdd(&b.flags[F_SKIN], 1);
    }
    // atoms beyond the grid extent of a free axis (clamped into edge cells)
    for (int a = 0; a < 3; ++a) {
        if (bx.pmask & (1 << a)) continue;
        const double xa = a == 0 ? x.x : (a == 1 ? x.y : x.z);
        const double f = (xa - bx.o[a]) * bx.iL[a];
        if (f < 0.0 || f >= 1.0) {
            atomicAdd(&b.flags[F_OUTSIDE], 1);
            break;
        }
    }
}

__global__ void k_bin(Buffers b, int p, int q, int64_t n_slots, double half_skin2, int check_skin,
                      const int32_t* __restrict__ gate)
{
    if (gate && gate[0] == 0) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = global_thread(); t < n_slots; t += stride)
        if (!replica_kept(b, gate, t)) bin_slot(b, p, q, t, half_skin2, check_skin);
}

// Rebuild stage 2: exclusive scan of cell populations, shifted into slot numbering
// with the per-cell replica shift.  The populations binned by stage 1 are taken over
// (a kept replica's cells keep theirs).  One kernel where no replica has more than
// kScanOnce cells, each block summing the populations before its own in the replica
// of its first cell; beyond, where the blocks' readings grow with the square of the
// cells, a block scan and a second kernel that adds the sums of the block totals
// before each block.  One kernel against two: 2000 atoms 2.0 and 9.4 us, 256 liquids
// 4.8 and 9.4, 138,000 cells of one replica 18.4 and 9.9.
constexpr int kScanBlock = 1024;
constexpr int32_t kScanOnce = 1 << 16;

// Inclusive sums over the wavefront.
__device__ __forceinline__ int32_t wave_inclusive_scan(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15, 31
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return v;
}

// Exclusive sums over the workgroup, and its total.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t& total)
{
    __shared__ int32_t part[kScanBlock / kWave];
    const int32_t incl = wave_inclusive_scan(v);
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) part[threadIdx.x / kWave] = incl;
    __syncthreads();
    int32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kScanBlock / kWave; ++w) {
        if (w < (int)(threadIdx.x / kWave)) before += part[w];
        total += part[w];
    }
    return before + incl - v;
}

// Sum of a value over the workgroup.
__device__ __forceinline__ int32_t block_sum(int32_t v)
{
    __shared__ int32_t sums[kScanBlock / kWave];
    const int32_t incl = wave_inclusive_scan(v);
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) sums[threadIdx.x / kWave] = incl;
    __syncthreads();
    int32_t all = 0;
#pragma unroll
    for (int w = 0; w < kScanBlock / kWave; ++w) all += sums[w];
    return all;
}

// Whether cell i belongs to a replica that keeps its list in this build.
__device__ __forceinline__ bool cell_kept(const Buffers& b, int64_t i, const int32_t* gate)
{
    if (!gate) return false;
    const int r = b.cell_rep[i];
    return r >= 0 && gate[1 + r] == 0;
}

__global__ __launch_bounds__(kScanBlock) void k_scan(Buffers b, int32_t n, const int32_t* __restrict__ gate)
{
    if (gate && gate[0] == 0) return;
    // Cells before this block, in the replica of its first cell (those of the
    // replicas before hold exactly their atoms; integers: any order is exact).
    const int64_t first = (int64_t)blockIdx.x * kScanBlock;
    const int r0 = b.cell_rep[first];
    int32_t run = 0;
    if (r0 >= 0) {
        const DevReplica& R = b.reps[r0];
        const int32_t* __restrict__ count = cell_kept(b, first, gate) ? b.cell_count : b.bin_count;
        if (threadIdx.x == 0) run = R.atom_off;
#pragma unroll 8
        for (int64_t k = R.cell_off + threadIdx.x; k < first; k += kScanBlock) run += count[k];
    }
    const int64_t i = first + threadIdx.x;
    int32_t v = 0;
    if (i < n) {
        if (cell_kept(b, i, gate)) {
            v = b.cell_count[i];
        } else {
            v = b.bin_count[i];  // (other blocks read it too: cleared by stage 3)
            b.cell_count[i] = v;
            b.cell_cursor[i] = 0;
        }
    }
    const int32_t before = block_sum(run);
    int32_t total;
    const int32_t ex = block_exclusive_scan(v, total);
    if (i < n) b.cell_start[i] = before + ex + b.cell_shift[i];
    if (gate && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&b.flags[F_AUTO_BUILDS], 1);
}

__global__ __launch_bounds__(kScanBlock) void k_scan_local(Buffers b, int32_t n, const int32_t* __restrict__ gate)
{
    if (gate && gate[0] == 0) return;
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    int32_t v = 0;
    if (i < n) {
        if (cell_kept(b, i, gate)) {
            v = b.cell_count[i];
        } else {
            v = b.bin_count[i];
            b.cell_count[i] = v;
            b.cell_cursor[i] = 0;
        }
    }
    int32_t total;
    const int32_t ex = block_exclusive_scan(v, total);
    if (i < n) b.cell_start[i] = ex;
    if (threadIdx.x == 0) b.scan_blocks[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_add(Buffers b, int32_t n, const int32_t* __restrict__ gate)
{
    if (gate && gate[0] == 0) return;
    int32_t run = 0;  // the totals of the blocks before this one
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += kScanBlock) run += b.scan_blocks[k];
    const int32_t before = block_sum(run);
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    if (i < n) b.cell_start[i] += before + b.cell_shift[i];
    if (gate && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(&b.flags[F_AUTO_BUILDS], 1);
}

// Rebuild stage 3: place every atom in its cell's slot range (arbitrary order within
// the cell, fixed by the next kernel), and clear the bins for the next build (a kept
// replica's are zero already).
__global__ void k_scatter(Buffers b, int64_t n_slots, int32_t n_cells, const int32_t* __restrict__ gate)
{
    if (gate && gate[0] == 0) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, first = global_thread();
    for (int64_t i = first; i < n_cells; i += stride) b.bin_count[i] = 0;
    for (int64_t t = first; t < n_slots; t += stride) {
        if (replica_kept(b, gate, t)) continue;
        const int c = b.cell_of[t];
        const int k = wave_run_add(b.cell_cursor, c);
        if (c >= 0) b.perm[b.cell_start[c] + k] = (int32_t)t;
    }
}

// Rebuild stage 4: order each cell's members by caller index, making the slot order
// (and so every later floating-point sum) independent of atomics' timing, and gather
// the whole atom state into that order.  Every member counts the members of its cell
// with a smaller caller index (indices are distinct): that count is its place in the
// cell, where its state goes.  (One kernel: the order has no use of its own, and the
// permuted slots are written and read once less; 1,013,760 atoms 15 + 48 -> 60 us, 2000 atoms 5.1 + 6.0 -> 8.6.)
__device__ __forceinline__ void gather_slot(const Buffers& b, int p, int q, int64_t u, int compact)
{
    const DevReplica& R = b.reps[uniform(b.rep_of_wave[u / kWave])];
    const int pn = p ^ 1, qn = q ^ 1;
    if (u - R.slot_off < R.n_atoms) {
        const int32_t t = b.perm[u];
        const int cell = b.cell_of[t];
        const double3 x = load_xyz(b.pos[p], t);
        const int beg = b.cell_start[cell], cnt = b.cell_count[cell];
        const int32_t* __restrict__ id = b.id[q];
        const int32_t key = id[t];
        int place = 0;
#pragma unroll 4
        for (int j = 0; j < cnt; ++j) place += id[b.perm[beg + j]] < key ? 1 : 0;
        const int64_t w = beg + place;  // the atom's new slot
        double xw[3] = {x.x, x.y, x.z};
        // re-wrap atoms that left the primary box on a periodic axis
        if (R.tri) {  // sheared cell: whole edge vectors, from the fractional coordinates
            double f[3];
            frac_coords(R.hinv, R.origin, xw[0], xw[1], xw[2], f);
            double k[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                k[a] = floor(f[a]);
                b.img[qn][a][w] = b.img[q][a][t] + (int32_t)k[a];
            }
            double sh[3];
            lattice_shift(R, k[0], k[1], k[2], sh);
#pragma unroll
            for (int a = 0; a < 3; ++a) xw[a] -= sh[a];
        } else {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                int32_t n = b.img[q][a][t];
                if (R.periodic_mask & (1 << a)) {
                    const double s = floor((xw[a] - R.origin[a]) * R.inv_box[a]);
                    if (s != 0.0) {
                        xw[a] -= s * R.box[a];
                        n += (int32_t)s;
                    }
                }
                b.img[qn][a][w] = n;
            }
        }
        const double4 x4 = make_double4(xw[0], xw[1], xw[2], 0.0);
        b.pos[pn][w] = x4;
        b.xbuild[w] = x4;
        if (compact) {
            // the slot's link cell and its compact record (here, where every lane
            // holds an atom, and not in the list kernel, whose wavefronts own a
            // handful each)
            const int cpk = b.cell_coord[cell];
            const int c[3] = {cpk & 1023, (cpk >> 10) & 1023, cpk >> 20};
            int4 rq;
            if (!compact_coords(R, c, xw[0], xw[1], xw[2], rq)) atomicAdd(&b.flags[F_COMPACT], 1);
            b.cellxyz[w] = make_int4(c[0], c[1], c[2], 0);
            b.rec[0][w] = rq;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) b.vel[qn][a][w] = b.vel[q][a][t];
        b.id[qn][w] = b.id[q][t];
        b.type[qn][w] = b.type[q][t];
        b.pwork[qn][w] = b.pwork[q][t];
        if (b.acc[q][0]) {  // Gear integrator state travels with its atom
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                b.acc[qn][a][w] = b.acc[q][a][t];
                b.jrk[qn][a][w] = b.jrk[q][a][t];
            }
        }
    } else {
        const double4 z = make_double4(0.0, 0.0, 0.0, 0.0);
        b.pos[pn][u] = z;
        b.xbuild[u] = z;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            b.vel[qn][a][u] = 0.0;
            b.img[qn][a][u] = 0;
        }
        b.id[qn][u] = -1;
        b.type[qn][u] = kEmptySlot;
        b.pwork[qn][u] = 0.0;
        if (b.acc[q][0]) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                b.acc[qn][a][u] = 0.0;
                b.jrk[qn][a][u] = 0.0;
            }
        }
    }
}

__global__ void k_gather(Buffers b, int p, int q, int64_t n_slots, int compact, const int32_t* __restrict__ gate)
{
    if (gate && gate[0] == 0) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t u = global_thread(); u < n_slots; u += stride)
        if (!replica_kept(b, gate, u)) gather_slot(b, p, q, u, compact);
}

// Verlet list from the link cells (paper, "The Neighbourlist calculation":
// each cell's atoms are tested against the atoms of the 27 cells around it).  One wavefront per link
// cell.  The up to 27 adjacent cells (fewer on free faces; on a periodic axis
// with under three cells each distinct cell once) become one candidate
// sequence: cell by cell (x fastest), atoms in slot order.  The wavefront
// holds up to 64 x kCandPasses candidates in registers, shifted by the periodic
// image of their cell, and tests every atom of its own cell against them;
// the in-range lanes of each test are packed with ballots, so list entries
// come out in candidate order, inner ones first.  Full list: every j != i with r < r_c + skin;
// half list: only j with a larger slot index.
//
// Entries: slot | code << kIndexBits, 2 bits per axis; a row's inner entries
// (pairs closer than r_d + skin) come first.  FP64 mode: the periodic image (0 none, 1 +L,
// 2 -L); compact mixed mode: the unwrapped link-cell offset plus one.  Axes with one or two periodic cells have no
// unique image per cell; there the image is the minimum one of each pair.
// Layout: groups of four entries per slot (nbr_at).  Overflow keeps counting, so the
// required capacity can be reported.
// Adjacency of every link cell, once per geometry: entry k of cell c is the
// cell at offset (k % 3 - 1, k / 3 % 3 - 1, k / 9 - 1), or -1 where a free
// face ends the grid or a periodic axis of under three cells would list a
// cell twice.  .y: periodic image of that cell (2 bits per axis, 1 = +L,
// 2 = -L) and, from bit 8, its unwrapped offset plus one.  On periodic axes
// with under three cells the image is left to the pair (minimum image) and
// the offset is the plain one between the two cells.
__global__ void k_cell_table(Buffers b, int32_t n_cells)
{
    const int64_t t = global_thread();
    if (t >= (int64_t)n_cells * 27) return;
    const int cell = (int)(t / 27), k = (int)(t - (int64_t)cell * 27);
    const int r = b.cell_rep[cell];
    if (r < 0) {
        b.cell_adj[t] = make_int2(-1, 0);
        if (k == 13) b.cell_coord[cell] = 0;
        return;
    }
    const DevReplica& R = b.reps[r];
    const int local = cell - R.cell_off;
    const int brick = local / R.cpb, in = local - brick * R.cpb;
    const int c[3] = {(brick % R.nbk[0]) * R.bd[0] + in % R.bd[0],
                      ((brick / R.nbk[0]) % R.nbk[1]) * R.bd[1] + (in / R.bd[0]) % R.bd[1],
                      (brick / (R.nbk[0] * R.nbk[1])) * R.bd[2] + in / (R.bd[0] * R.bd[1])};
    const int o[3] = {k % 3 - 1, (k / 3) % 3 - 1, k / 9 - 1};
    bool ok = true;
    int cc[3], wrap = 0, code = 0;
    for (int a = 0; a < 3; ++a) {
        int v = c[a] + o[a], w = 0;
        ok = ok && c[a] < R.nc[a];  // padding cells of the brick grid have no atoms
        if (R.periodic_mask >> a & 1) {
            if (R.nc[a] == 1) ok = ok && o[a] == 0;
            if (R.nc[a] == 2) ok = ok && o[a] >= 0;
            if (v < 0) v += R.nc[a], w = 2;
            if (v >= R.nc[a]) v -= R.nc[a], w = 1;
        } else {
            ok = ok && v >= 0 && v < R.nc[a];
        }
        cc[a] = v;
        const bool few = (R.periodic_mask >> a & 1) && R.nc[a] < 3;
        wrap |= (few ? 0 : w) << (2 * a);
        code |= (few ? v - c[a] + 1 : o[a] + 1) << (2 * a);
    }
    b.cell_adj[t] = make_int2(ok ? cell_index(R, cc[0], cc[1], cc[2]) : -1, wrap | (code << 8));
    if (k == 13) b.cell_coord[cell] = c[0] | (c[1] << 10) | (c[2] << 20);
}

constexpr int kCandPasses = 4;  // sets of 64 candidates held in registers at most

__device__ __forceinline__ double select_shift(int s, double L) { return s == 1 ? L : (s == 2 ? -L : 0.0); }

// Moves a candidate by the periodic image of its cell.
template <bool TRI>
__device__ __forceinline__ void candidate_shift(const Box& bx, int w, double3& x)
{
    if (TRI) {
        double d[3] = {0.0, 0.0, 0.0};
        apply_shift(bx, w, d[0], d[1], d[2]);
        x.x += d[0];
        x.y += d[1];
        x.z += d[2];
    } else {
        x.x += select_shift(w & 3, bx.L[0]);
        x.y += select_shift((w >> 2) & 3, bx.L[1]);
        x.z += select_shift((w >> 4) & 3, bx.L[2]);
    }
}


// Minimum image of one pair along the axes in `amb` (periodic axes with fewer
// than three cells), with the entry's code field updated: the image shift in
// FP64 mode, the unwrapped link-cell offset plus one in compact mode.
__device__ __forceinline__ void min_image_axis(double& d, double L, double iL, int nc, int a, int compact, int& e)
{
    const double s = rint(d * iL);
    d -= s * L;
    const int sh = kIndexBits + 2 * a;
    const int f = (e >> sh) & 3;
    const int nf = compact ? f - (int)s * nc : (s < 0.0 ? 1 : (s > 0.0 ? 2 : 0));
    e = (e & ~(3 << sh)) | (nf << sh);
}

__device__ __forceinline__ void min_image_pair(const Box& bx, int amb, int compact, double& dx, double& dy, double& dz,
                                               int& e)
{
    if (amb & 1) min_image_axis(dx, bx.L[0], bx.iL[0], bx.nc[0], 0, compact, e);
    if (amb & 2) min_image_axis(dy, bx.L[1], bx.iL[1], bx.nc[1], 1, compact, e);
    if (amb & 4) min_image_axis(dz, bx.L[2], bx.iL[2], bx.nc[2], 2, compact, e);
}

// Where the list build writes.  Lists below 4 GiB are written through raw
// buffer resources: the atom's row start is a scalar byte offset and each lane
// adds its entry's 32-bit offset, so the address costs three vector
// instructions; WIDE lists take 64-bit addresses.  With several species each
// entry also gets its neighbour's type byte, in the same layout (four bytes
// per group of four entries), so the force loop reads them with its entries
// instead of gathering them one by one.
struct ListOut {
    __amdgpu_buffer_rsrc_t rs, ts;  // entries, type bytes
    uint32_t group_bytes;           // n_slots * 16: one group of four entries of every slot
    int32_t* nbr;
    uint8_t* types;
    int64_t n_slots;
};


// What a wavefront of the list build works on: one chunk of own atoms and the
// candidates it tests them against.
struct ListWork {
    const double4* pos;
    const uint8_t* type;    // of the candidates' slots
    const int2* tab;        // candidate -> {slot, image and offset codes}
    const uint16_t* kept;   // the candidates that remain, as table indices (pruned)
    int n_cand;             // candidates to test
    int s0, n;              // own atoms s0 .. s0 + n - 1; lane l holds atom s0 + l in xl
    double3 xl;
    int32_t cap;
    double rlist2, rdl2;
    int half_list, compact, amb;
    bool tabled, pruned, any_wrap;
    int excl, nb_start, nb_wrap, nb_code;  // lane k: adjacent cell k (without the table)
};

// Tests the own atoms against NP sets of 64 candidates from candidate g0 on, held
// in registers, and appends the in-range ones to the atoms' rows.
//
// SPLIT: a row holds its inner entries (closer than r_d + skin) first, then the
// others, each in candidate order.  All sets are tested before an entry is
// stored, so with every candidate in registers (ONCE) the place behind the inner
// entries is known in time; otherwise a COUNT sweep over all candidates comes
// first and `my_outer` enters as that place.  On return lane l's `my_inner` is
// the number of inner entries of its atom so far and `my_outer` the place behind
// its last entry.
template <int NP, bool TRI, bool AMB, bool WIDE, bool SPLIT, bool WT, bool COUNT, bool ONCE>
__device__ __forceinline__ void test_candidates(const ListOut& L, const ListWork& W, const Box& bx, int g0,
                                                int& my_inner, int& my_outer)
{
    const int lane = threadIdx.x & (kWave - 1);
    double cx[NP], cy[NP], cz[NP];
    int ce[NP], cj[NP], ct[NP];
    bool live[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int m0 = g0 + u * kWave + lane;
        int m = min(m0, W.n_cand - 1);
        int j, w, code;
        if (ONCE || W.tabled) {
            if (W.pruned) m = W.kept[m];
            const int2 tv = W.tab[m];
            j = tv.x;
            w = tv.y & 63;
            code = (tv.y >> 8) & 63;
        } else {
            // the adjacent cell holding candidate m: the last k with excl_k <= m
            int k = 0;
#pragma unroll
            for (int step = kWave / 2; step > 0; step >>= 1)
                if (__shfl(W.excl, k + step, kWave) <= m) k += step;
            j = __shfl(W.nb_start, k, kWave) + (m - __shfl(W.excl, k, kWave));
            w = __shfl(W.nb_wrap, k, kWave);
            code = __shfl(W.nb_code, k, kWave);
        }
        double3 xj = load_xyz(W.pos, j);
        if (W.any_wrap) candidate_shift<TRI>(bx, w, xj);
        cx[u] = xj.x;
        cy[u] = xj.y;
        cz[u] = xj.z;
        ce[u] = j | (code << kIndexBits);
        cj[u] = j;
        ct[u] = WT ? W.type[j] : 0;
        live[u] = m0 < W.n_cand;
    }
    // j != i (full list) or j > i (half list) as one unsigned compare of j - i - 1
    const uint32_t lim = W.half_list ? 0x7FFFFFFFu : 0xFFFFFFFFu;
    for (int ii = 0; ii < W.n; ++ii) {
        const int i = W.s0 + ii;
        const double xi = bcast_lane(W.xl.x, ii), yi = bcast_lane(W.xl.y, ii), zi = bcast_lane(W.xl.z, ii);
        bool take[NP], in[NP];
        int e[NP], n_inner = 0;
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            double dx = cx[u] - xi, dy = cy[u] - yi, dz = cz[u] - zi;
            e[u] = ce[u];
            if (AMB) min_image_pair(bx, W.amb, W.compact, dx, dy, dz, e[u]);
            const double r2 = dx * dx + dy * dy + dz * dz;
            take[u] = live[u] & ((uint32_t)(cj[u] - (i + 1)) < lim) & (r2 < W.rlist2);
            in[u] = SPLIT && (take[u] & (r2 < W.rdl2));
            if (SPLIT) n_inner += __popcll(__builtin_amdgcn_ballot_w64(in[u]));
        }
        if (COUNT) {
            if (lane == ii) my_inner += n_inner;
            continue;
        }
        int base_in = ONCE ? 0 : __builtin_amdgcn_readlane(my_inner, ii);
        int base_out = ONCE ? n_inner : __builtin_amdgcn_readlane(my_outer, ii);
        const uint32_t row = (uint32_t)i * 16u;  // entry k of atom i: row + (k / 4) group_bytes + 4 (k % 4)
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const uint64_t inner = SPLIT ? __builtin_amdgcn_ballot_w64(in[u]) : 0;
            const uint64_t outer = __builtin_amdgcn_ballot_w64(take[u]) & ~inner;
            // the lane's place among its kind
            const int k_out = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(outer >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)outer, base_out));
            int at_row = k_out;
            if (SPLIT) {
                const int k_in = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(inner >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)inner, base_in));
                at_row = in[u] ? k_in : k_out;
            }
            if (take[u] & (at_row < W.cap)) {
                const uint32_t k = (uint32_t)at_row;  // entry k of atom i (the layout of nbr_at)
                if (WIDE) {
                    const int64_t at = nbr_at(at_row, i, L.n_slots);
                    L.nbr[at] = e[u];
                    if (WT) L.types[at] = (uint8_t)ct[u];
                } else {
                    const uint32_t off = (k >> 2) * L.group_bytes + ((k & 3u) << 2);
                    __builtin_amdgcn_raw_buffer_store_b32(e[u], L.rs, off, row, 0);
                    if (WT)  // byte offsets a quarter of the entry's
                        __builtin_amdgcn_raw_buffer_store_b8((unsigned char)ct[u], L.ts, off >> 2, row >> 2, 0);
                }
            }
            base_in += __popcll(inner);
            base_out += __popcll(outer);
        }
        if (lane == ii) {
            my_inner = base_in;
            my_outer = base_out;
        }
    }
}

// Smallest values of the wavefront's lanes 0 .. n - 1 (the lanes beyond repeat
// one of those): within rows of 16 lanes by shifts, then, for n > 16, across the
// rows; a lane without a source keeps its value.  Written as one block of DPP
// minima, one instruction per step and value (the builtins take four: a move,
// two quieting maxima, the minimum); a value is read five instructions after it
// was written, beyond the two wait states DPP asks for.  The compiler does not see
// into a block, so each also waits at its ends: two states before its first DPP
// read, one after its last write, which a lane read may follow at once.
__device__ __forceinline__ void wave_min(float (&v)[6], int n)
{
#define MDK_DPP_STEP(ctrl)                      \
    "v_min_f32_dpp %0, %0, %0 " ctrl "\n\t"     \
    "v_min_f32_dpp %1, %1, %1 " ctrl "\n\t"     \
    "v_min_f32_dpp %2, %2, %2 " ctrl "\n\t"     \
    "v_min_f32_dpp %3, %3, %3 " ctrl "\n\t"     \
    "v_min_f32_dpp %4, %4, %4 " ctrl "\n\t"     \
    "v_min_f32_dpp %5, %5, %5 " ctrl "\n\t"
    asm volatile("s_nop 1\n\t"  // values just written
                 MDK_DPP_STEP("row_shr:1 row_mask:0xf bank_mask:0xf")
                 MDK_DPP_STEP("row_shr:2 row_mask:0xf bank_mask:0xf")
                 MDK_DPP_STEP("row_shr:4 row_mask:0xf bank_mask:0xf")
                 MDK_DPP_STEP("row_shr:8 row_mask:0xf bank_mask:0xf")
                 "s_nop 0"
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]));
    int last = 15;  // lane 15 of a row holds its minimum
    if (n > 16) {
        asm volatile("s_nop 1\n\t"
                     MDK_DPP_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf")
                     MDK_DPP_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf")
                     "s_nop 0"
                     : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]));
        last = kWave - 1;
    }
#undef MDK_DPP_STEP
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[k]), last));
}

// Inclusive sums over the first 32 lanes (lanes 27 .. 31 hold zeros here).
__device__ __forceinline__ int scan32(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into the next row
    return v;
}

// Largest list length over the wavefront, one atomic per wavefront.
__device__ __forceinline__ void wave_max_flag(int v, int32_t* flag)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, kWave));
    // The flag only grows, so a plain (possibly stale) read filters out the
    // atomics that cannot raise it: a kernel with many wavefronts would
    // otherwise serialise on one address.
    if ((threadIdx.x & (kWave - 1)) == 0 && v > 0 && v > *flag) atomicMax(flag, v);
}

// TRI: sheared cells (candidate shifts are edge-vector sums), a separate
// instantiation so the orthorhombic build keeps its short candidate loop.
// SPLIT: the inner entries (r < r_d + skin) of a row come first; otherwise every
// entry is inner.
// WT: several species (each entry's type byte is stored beside it).
// gate: the automatic rebuild's replica flags (NULL: every replica).
// copy_back: also copy each own atom's sorted state from (p, q) into
// (p ^ 1, q ^ 1), the buffers an automatic rebuild keeps using.
template <bool TRI, bool WIDE, bool SPLIT, bool WT>
__device__ __forceinline__ void list_cell(const Buffers& b, int p, int q, int64_t n_slots, int cell, int32_t cap,
                                          double rlist2, double rdl2, int half_list, int compact,
                                          const int32_t* __restrict__ gate, int copy_back)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int r = uniform(b.cell_rep[cell]);
    if (r < 0) return;
    if (gate && gate[1 + r] == 0) return;
    const int n_own = uniform(b.cell_count[cell]);
    if (n_own == 0) return;
    const int s_own = uniform(b.cell_start[cell]);
    const int seen = b.flags[F_MAX_COUNT];  // (read early, or its latency would end every wavefront)
    const DevReplica& R = b.reps[r];
    const Box bx = load_box(R);
    int amb = 0;  // periodic axes with fewer than three cells
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if ((bx.pmask >> a & 1) && bx.nc[a] < 3) amb |= 1 << a;

    // lane k < 27: adjacent cell k
    int nb_start = 0, nb_count = 0, nb_wrap = 0, nb_code = 0;
    if (lane < 27) {
        const int2 adj = b.cell_adj[(int64_t)cell * 27 + lane];
        nb_wrap = adj.y & 63;
        nb_code = compact ? (adj.y >> 8) & 63 : nb_wrap;
        if (adj.x >= 0) {
            nb_start = b.cell_start[adj.x];
            nb_count = b.cell_count[adj.x];
        }
    }
    // whether any adjacent cell lies across a face (interior cells, most of a
    // large box, skip the candidates' shifts)
    const bool any_wrap = __ballot(nb_wrap != 0) != 0;
    // exclusive prefix of the candidate counts over the 27 lanes
    const int incl = scan32(nb_count);
    const int excl = lane < 27 ? incl - nb_count : INT32_MAX;  // (lanes beyond never start at a candidate)
    const int total = __builtin_amdgcn_readlane(incl, 26);

    // candidate table of this wave: slot and codes of candidate m, written by
    // the 27 lanes of the adjacent cells (lane k its own cell's run), read back
    // by candidate index.  A wave's LDS operations complete in order, so the
    // wave-scope fence suffices.  Larger stencils search the prefix instead.
    __shared__ int2 cand_table[kBlock / kWave][kCandTable];
    int2* tab = cand_table[threadIdx.x / kWave];
    const bool tabled = total <= kCandTable;
    if (tabled) {
        const int wc = nb_wrap | (nb_code << 8);
        for (int qq = 0; qq < nb_count; ++qq) tab[excl + qq] = make_int2(nb_start + qq, wc);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // the candidates that remain for a chunk of own atoms, as table indices
    __shared__ uint16_t kept_table[kBlock / kWave][kCandTable];
    uint16_t* kept = kept_table[threadIdx.x / kWave];
    const float rlist = sqrtf((float)rlist2), prune = rlist + (1e-3f + 1e-6f * rlist);
    const float prune2 = prune * prune;

    const double4* __restrict__ pos = b.pos[p];
    // (WIDE: the buffer resources are unused; their sizes wrap harmlessly)
    ListOut L;
    L.group_bytes = (uint32_t)n_slots * 16u;
    const uint32_t n_groups = (uint32_t)((cap + 2 * kChunk - 1) / kChunk);
    L.rs = __builtin_amdgcn_make_buffer_rsrc(b.nbr, (short)0, (int)(L.group_bytes * n_groups), (int)kBufferWord3);
    L.ts = __builtin_amdgcn_make_buffer_rsrc(b.ntype, (short)0, (int)(L.group_bytes / 4 * n_groups), (int)kBufferWord3);
    L.nbr = b.nbr;
    L.types = b.ntype;
    L.n_slots = n_slots;
    for (int i0 = 0; i0 < n_own; i0 += kWave) {
        const int n_chunk = min(kWave, n_own - i0);
        // lane l holds atom s_own + i0 + l; the test loop broadcasts it
        const double3 xl = load_xyz(pos, s_own + i0 + min(lane, n_chunk - 1));
        ListWork W = {pos, b.type[q], tab, kept, total, s_own + i0, n_chunk, xl, cap, rlist2, rdl2, half_list, compact, amb,
                      tabled, false, any_wrap, excl, nb_start, nb_wrap, nb_code};
        // Candidates beyond the list radius of the box around these atoms are
        // left out first (in FP32 relative to the first own atom, with a margin
        // of 0.001 A + 1e-6 of the radius: where the box is below 1000 A wide, the
        // candidates near the limit are rounded by 6e-5 A + 6e-8 of the radius per
        // step; not where pairs take their minimum image one by one).  The tests, ~20 vector instructions per own
        // atom and 64 candidates, bound this kernel, and about half of the 27
        // cells' candidates go.  It pays from ~10 atoms per cell: Fe-C replicas
        // at a 0.8 A skin 211 -> 157 us per build with the gather, the fcc slab
        // 120 -> 95, sheared 128,000 atoms 81 -> 60.  At 7 atoms per cell it costs about
        // what it saves (without it every build is 1 to 4% slower still), and the order
        // of the rows comes on top: whole builds against those of unordered rows, 1,013,760
        // atoms FP64 363 -> 364 us and mixed 377 -> 395, 2,635,380 atoms 942 -> 970 and 959
        // -> 1009.  A step that uses the list has it back in its density pass (mixed 56 ->
        // 42); with a build at every step mixed loses 1.5% at the former size (486 -> 494).
        if (tabled && amb == 0) {
            const double xr = bcast_lane(xl.x, 0), yr = bcast_lane(xl.y, 0), zr = bcast_lane(xl.z, 0);
            const float ox = (float)(xl.x - xr), oy = (float)(xl.y - yr), oz = (float)(xl.z - zr);
            float lo[6] = {ox, oy, oz, -ox, -oy, -oz};
            wave_min(lo, n_chunk);
            const float hx = -lo[3], hy = -lo[4], hz = -lo[5];
            if (hx - lo[0] < 1000.0f && hy - lo[1] < 1000.0f && hz - lo[2] < 1000.0f) {
                int n_cand = 0;
                for (int g0 = 0; g0 < total; g0 += 2 * kWave) {
                    float px[2], py[2], pz[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {  // both loads before the first test
                        const int m0 = g0 + u * kWave;
                        if (m0 >= total) continue;
                        const int2 tv = tab[min(m0 + lane, total - 1)];
                        double3 xj = load_xyz(pos, tv.x);
                        if (any_wrap) candidate_shift<TRI>(bx, tv.y & 63, xj);
                        px[u] = (float)(xj.x - xr);
                        py[u] = (float)(xj.y - yr);
                        pz[u] = (float)(xj.z - zr);
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int m0 = g0 + u * kWave;
                        if (m0 >= total) continue;
                        const float ex = fmaxf(fmaxf(lo[0] - px[u], px[u] - hx), 0.0f),
                                    ey = fmaxf(fmaxf(lo[1] - py[u], py[u] - hy), 0.0f),
                                    ez = fmaxf(fmaxf(lo[2] - pz[u], pz[u] - hz), 0.0f);
                        const bool keep = m0 + lane < total && fmaf(ex, ex, fmaf(ey, ey, ez * ez)) <= prune2;
                        const uint64_t mask = __builtin_amdgcn_ballot_w64(keep);
                        const int at = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)mask, n_cand));
                        if (keep) kept[at] = (uint16_t)(m0 + lane);
                        n_cand += __popcll(mask);
                    }
                }
                W.n_cand = n_cand;
                W.pruned = true;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
        // lane l: inner entries of that atom so far, and the place behind its others
        int my_inner = 0, my_outer = 0;
        if (W.pruned && W.n_cand <= kWave * kCandPasses) {
            if (W.n_cand <= kWave) test_candidates<1, TRI, false, WIDE, SPLIT, WT, false, true>(L, W, bx, 0, my_inner, my_outer);
            else if (W.n_cand <= 2 * kWave)
                test_candidates<2, TRI, false, WIDE, SPLIT, WT, false, true>(L, W, bx, 0, my_inner, my_outer);
            else if (W.n_cand <= 3 * kWave)
                test_candidates<3, TRI, false, WIDE, SPLIT, WT, false, true>(L, W, bx, 0, my_inner, my_outer);
            else test_candidates<4, TRI, false, WIDE, SPLIT, WT, false, true>(L, W, bx, 0, my_inner, my_outer);
        } else {
            if (SPLIT) {  // count the inner entries; the others go behind them
                for (int g0 = 0; g0 < W.n_cand; g0 += 2 * kWave)
                    if (amb) test_candidates<2, TRI, true, WIDE, SPLIT, WT, true, false>(L, W, bx, g0, my_inner, my_outer);
                    else test_candidates<2, TRI, false, WIDE, SPLIT, WT, true, false>(L, W, bx, g0, my_inner, my_outer);
                my_outer = my_inner;
                my_inner = 0;
            }
            for (int g0 = 0; g0 < W.n_cand; g0 += 2 * kWave)
                if (amb) test_candidates<2, TRI, true, WIDE, SPLIT, WT, false, false>(L, W, bx, g0, my_inner, my_outer);
                else test_candidates<2, TRI, false, WIDE, SPLIT, WT, false, false>(L, W, bx, g0, my_inner, my_outer);
        }
        const int my_count = my_outer;
        // per-atom epilogue: counts, overflow flag
        const int i = s_own + i0 + lane;
        if (lane < n_chunk) {
            b.ncount[i] = min(my_count, cap);
            b.ninner[i] = min(SPLIT ? my_inner : my_count, cap);
            if (copy_back) {  // (no lane of this kernel reads the buffers written here)
                const int pn = p ^ 1, qn = q ^ 1;
                b.pos[pn][i] = pos[i];
                b.id[qn][i] = b.id[q][i];
                b.type[qn][i] = b.type[q][i];
                b.pwork[qn][i] = b.pwork[q][i];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    b.vel[qn][a][i] = b.vel[q][a][i];
                    b.img[qn][a][i] = b.img[q][a][i];
                }
                if (b.acc[q][0]) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        b.acc[qn][a][i] = b.acc[q][a][i];
                        b.jrk[qn][a][i] = b.jrk[q][a][i];
                    }
                }
            }
        }
        if (__builtin_amdgcn_ballot_w64(lane < n_chunk && my_count > seen) != 0)
            wave_max_flag(lane < n_chunk ? my_count : 0, &b.flags[F_MAX_COUNT]);
    }
}

// One wavefront per link cell.  LOOP (gated builds): a capped grid, each
// wavefront taking every `waves`-th cell (a wavefront's LDS operations
// complete in order, so its candidate table is simply refilled for the next
// cell); a separate instantiation, since the loop keeps more registers live.
template <bool TRI, bool WIDE, bool SPLIT, bool WT, bool LOOP>
__global__ __launch_bounds__(kBlock, TRI ? 4 : LOOP ? 5 : 6) void k_cell_list(Buffers b, int p, int q, int64_t n_slots, int32_t n_cells,
                                                      int32_t cap, double rlist2, double rdl2, int half_list,
                                                      int compact, const int32_t* __restrict__ gate, int copy_back)
{
    const int64_t w0 = logical_block() * (kBlock / kWave) + threadIdx.x / kWave;
    if (!LOOP) {
        if (w0 < n_cells)
            list_cell<TRI, WIDE, SPLIT, WT>(b, p, q, n_slots, uniform((int)w0), cap, rlist2, rdl2, half_list,
                                            compact, nullptr, 0);
        return;
    }
    if (gate[0] == 0) return;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t w = w0; w < n_cells; w += waves)
        list_cell<TRI, WIDE, SPLIT, WT>(b, p, q, n_slots, uniform((int)w), cap, rlist2, rdl2, half_list, compact,
                                        gate, copy_back);
}

}  // namespace

void launch_rebuild(const Buffers& b, int p, int q, const KernelShape& k, double half_skin2, const int32_t* gate,
                    hipStream_t s)
{
    // p, q: current buffers; the sorted state lands in p^1, q^1.  The cell
    // populations are binned into bin_count, which every build leaves zeroed.
    const int64_t slot_blocks = gate ? std::min<int64_t>(blocks_for(k.n_slots), kGatedBlocks) : blocks_for(k.n_slots);
    hipLaunchKernelGGL(k_bin, dim3(slot_blocks), dim3(kBlock), 0, s, b, p, q, k.n_slots,
                       half_skin2, half_skin2 >= 0.0 ? 1 : 0, gate);
    const int nb = (int)((k.n_cells + kScanBlock - 1) / kScanBlock);
    if (k.rep_cells <= kScanOnce) {
        hipLaunchKernelGGL(k_scan, dim3(nb), dim3(kScanBlock), 0, s, b, k.n_cells, gate);
    } else {
        hipLaunchKernelGGL(k_scan_local, dim3(nb), dim3(kScanBlock), 0, s, b, k.n_cells, gate);
        hipLaunchKernelGGL(k_scan_add, dim3(nb), dim3(kScanBlock), 0, s, b, k.n_cells, gate);
    }
    hipLaunchKernelGGL(k_scatter, dim3(slot_blocks), dim3(kBlock), 0, s, b, k.n_slots, k.n_cells, gate);
    hipLaunchKernelGGL(k_gather, dim3(slot_blocks), dim3(kBlock), 0, s, b, p, q, k.n_slots, k.compact, gate);
}

// Displacement check of the automatic rebuild: the same criterion as the skin
// guard of scheduled builds (no atom may move more than skin/2 between builds
// for a list of r_c + skin to hold every pair closer than r_c), tested at every
// step before the list is used, per replica.  Block 0 also clears the flag set
// of the next check (the rebuild kernels of the previous check, its readers,
// ran before this kernel).
__global__ void k_skin_check(Buffers b, int p, int64_t n_slots, int32_t n_rep, double guard2,
                             int32_t* __restrict__ gate, int32_t* __restrict__ next)
{
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i <= n_rep; i += blockDim.x) next[i] = 0;
    const int64_t t = global_thread();
    if (t >= n_slots) return;
    const double3 x = load_xyz(b.pos[p], t);
    const double3 x0 = load_xyz(b.xbuild, t);  // (empty slots: both zero)
    const double dx = x.x - x0.x, dy = x.y - x0.y, dz = x.z - x0.z;
    const bool far = fma(dx, dx, fma(dy, dy, dz * dz)) > guard2;
    if (__ballot(far) != 0 && (threadIdx.x & (kWave - 1)) == 0) {
        atomicOr(&gate[1 + b.rep_of_wave[t / kWave]], 1);
        atomicOr(&gate[0], 1);
    }
}

void launch_skin_check(const Buffers& b, int p, const KernelShape& k, double guard2, int32_t* gate,
                       int32_t* next, hipStream_t s)
{
    hipLaunchKernelGGL(k_skin_check, dim3(blocks_for(k.n_slots)), dim3(kBlock), 0, s, b, p, k.n_slots,
                       k.n_replicas, guard2, gate, next);
}

void launch_build_list(const Buffers& b, int p, int q, const KernelShape& k, double rlist2, double rdl2,
                       int half_list, const int32_t* gate, int copy_back, hipStream_t s)
{
    int64_t blocks = ((int64_t)k.n_cells + kBlock / kWave - 1) / (kBlock / kWave);
    if (gate) blocks = std::min<int64_t>(blocks, kGatedBlocks * 5 / 8);
    const bool wide = (uint64_t)k.n_slots * 16 * (uint64_t)((k.cap + 2 * kChunk - 1) / kChunk) >= ((uint64_t)1 << 32);
    const bool split = !half_list && rdl2 < rlist2;
    const int which = (k.tri ? 8 : 0) | (wide ? 4 : 0) | (split ? 2 : 0) | (k.list_types ? 1 : 0);
    using Kern = void (*)(Buffers, int, int, int64_t, int32_t, int32_t, double, double, int, int, const int32_t*, int);
    // [gated][TRI WIDE SPLIT WT]
    static const Kern kerns[2][16] = {
#define MDK_LIST_ROW(G)                                                                                             \
    {k_cell_list<false, false, false, false, G>, k_cell_list<false, false, false, true, G>,                        \
     k_cell_list<false, false, true, false, G>,  k_cell_list<false, false, true, true, G>,                         \
     k_cell_list<false, true, false, false, G>,  k_cell_list<false, true, false, true, G>,                         \
     k_cell_list<false, true, true, false, G>,   k_cell_list<false, true, true, true, G>,                          \
     k_cell_list<true, false, false, false, G>,  k_cell_list<true, false, false, true, G>,                         \
     k_cell_list<true, false, true, false, G>,   k_cell_list<true, false, true, true, G>,                          \
     k_cell_list<true, true, false, false, G>,   k_cell_list<true, true, false, true, G>,                          \
     k_cell_list<true, true, true, false, G>,    k_cell_list<true, true, true, true, G>}
        MDK_LIST_ROW(false), MDK_LIST_ROW(true)};
#undef MDK_LIST_ROW
    hipLaunchKernelGGL(kerns[gate ? 1 : 0][which], dim3(blocks), dim3(kBlock), 0, s, b, p, q, k.n_slots, k.n_cells,
                       k.cap, rlist2, half_list ? rlist2 : rdl2, half_list, k.compact, gate, copy_back);
}

void launch_cell_table(const Buffers& b, const KernelShape& k, hipStream_t s)
{
    hipLaunchKernelGGL(k_cell_table, dim3(blocks_for((int64_t)k.n_cells * 27)), dim3(kBlock), 0, s, b, k.n_cells);
}

}  // namespace mdk
