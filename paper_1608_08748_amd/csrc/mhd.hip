// Host runtime and C ABI (include/mhdchem.h) of the HIP implementation of one
// operator-split step of ideal MHD with H/H2 chemistry on a uniform periodic
// grid (Kulikov, Chernykh & Protasov, arXiv:1608.08748), for AMD MI355X.
//
// Stage names: NONADV is the paper's "eulerian" stage (Sec. 2.4, 2.5: pressure,
// Lorentz force, p dV work, face-field update); ADV is its "lagrangian" stage
// (Sec. 2.6: advection).
//
// Data layout in HBM: structure of arrays, one array of n cells per field,
// x fastest.  The state is split into three groups that are updated by
// different stages, each with three Runge-Kutta slots:
//   H = (rho, h2)            updated by ADV and the tail
//   M = (mx, my, mz, E, e)   updated by NONADV, ADV and the tail
//   B = (bx, by, bz)         updated by NONADV (face-centred, lower faces)
// so no stage copies a field it does not change.
//
// A step is a fixed program of kernel launches (mhd_kernels.hpp).  One box
// sends the program to its stream; the server runs the same program for every
// box in flight and merges the launches (one launch per program position over
// all boxes), so a box gets the same bits alone or in a batch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <deque>
#include <list>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <unordered_map>
#include <vector>

#include "mhd_kernels.hpp"
#include "mhdchem.h"

static_assert(mhd::NF == MHD_NFIELDS, "conserved field count of the kernels and the C ABI");

using namespace mhd;

// ---------------------------------------------------------------- box

// launches whose event pairs the timing ring holds (a step makes at most a
// few dozen)
constexpr int EVCAP = 1024;

// Pinned slots through which states leave for the caller's pageable memory
// (copy_out), allocated at the first use and released with their owner: an
// eighth of the state each, at most 4 MiB.
constexpr int RING_SLOTS = 8;
constexpr size_t RING_SLOT_MAX = (size_t)4 << 20;
struct HostRing {
    char* mem = nullptr;        // RING_SLOTS slots, then the fault flags
    size_t slot = 0;            // bytes per slot
    hipEvent_t ev[RING_SLOTS];
    int nev = 0;
};

struct mhd_box {
    mhd_params p;
    Geo g;
    hipStream_t s;
    int prec;          // MHD_FP64 / MHD_FP32_MIXED
    size_t esz;        // bytes per stored value
    int nblocks;       // cell-parallel blocks of NTH threads
    char* slot[3];     // three Runge-Kutta copies of the NF fields
    char* F[3];        // per-direction face outputs, 7 x N each (8 x N with the ionisation network)
    double* part;      // per-block partials: NF x nblocks
    uint32_t* flags;
    double* dt_dev;
    double* tot_dev;
    int grav;          // self-gravity on
    char* phi;         // gravitational potential, N values
    char* tw[3];       // per-axis FFT twiddles (n complex values)
    double* sf[3];     // per-axis 27-point stencil factors (n values)
    int cur[3];        // current slot of the groups H, M, B
    // cells per segment of the marching kernels (march_segments): the NONADV
    // faces along y and z, the ADV faces along y, the fused ADV update and the
    // face-field update along z
    int seg_fy, seg_fz, seg_ay, seg_xz, seg_b;
    bool stream;       // kernel outputs go past the caches (streamed())
    // per-launch event timing (mhd_set_timing)
    int timing;
    int nev;
    hipEvent_t ev[2 * EVCAP];
    int evcls[EVCAP], evparts[EVCAP];
    int ev_ready;
    double tms[MHD_NKCLASS];
    int64_t tcnt[MHD_NKCLASS];
    HostRing ring;
};

namespace {

enum { GH = 0, GM = 1, GB = 2 };
int group_of(int f)
{
    if (f == RHO || f == H2 || f == HP) return GH;
    if (f >= BX && f <= BZ) return GB;
    return GM;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
    size_t slot, F, part, misc, grav, total;
};

bool pow2_upto(int n, int cap) { return n >= 1 && n <= cap && (n & (n - 1)) == 0; }

// the FFT Poisson solve handles power-of-two axes up to 1024 cells
constexpr int FFT_MAX = 1024;

bool valid_physics(int32_t precision, double gamma, double cfl, double theta, int32_t chem, int32_t cool,
                   double nu, double Tu, double tu)
{
    if (!(gamma > 1.0) || !std::isfinite(gamma)) return false;
    if (!(cfl > 0.0) || !std::isfinite(cfl)) return false;
    if (!(theta >= 0.0) || !std::isfinite(theta)) return false;
    if (precision != MHD_FP64 && precision != MHD_FP32_MIXED) return false;
    if (chem != 0 && chem != 1) return false;
    if (cool != 0 && cool != 1) return false;
    if ((chem || cool) && !(nu > 0.0 && Tu > 0.0 && tu > 0.0)) return false;
    return true;
}

bool valid_dims(const int32_t n[3])
{
    for (int d = 0; d < 3; d++)
        if (n[d] < 1) return false;
    double c = (double)n[0] * n[1] * n[2];
    return c < 2147483647.0;
}

bool valid_params(const mhd_params* p)
{
    if (!p || !valid_dims(p->n)) return false;
    if (p->ionisation != 0 && p->ionisation != 1) return false;
    if (p->ionisation && !(p->n_unit_cm3 > 0.0 && p->T_unit_K > 0.0 && p->t_unit_s > 0.0)) return false;
    if (!(p->grav_G >= 0.0) || !std::isfinite(p->grav_G)) return false;
    if (p->grav_G > 0.0)
        for (int d = 0; d < 3; d++)
            if (!pow2_upto(p->n[d], FFT_MAX)) return false;
    return valid_physics(p->precision, p->gamma, p->cfl, p->theta, p->chemistry, p->cooling, p->n_unit_cm3,
                         p->T_unit_K, p->t_unit_s);
}

// face outputs per direction: 7 NONADV values, or 8 ADV fluxes with the
// ionisation network
size_t face_values(bool ion) { return ion ? NFACE + 1 : NFACE; }

void march_segments(mhd_box* b, double share);

// whether a launch over fields of this many bytes streams its outputs: the
// step's arrays together (about 54 fields) then hold the 256 MB Infinity Cache
// several times.  Level at 120^3 FP64 (13.8 MB) and between 128^3 (8.4 MB, 1.5%
// slower) and 144^3 FP32 (11.9 MB, 1% faster).
bool streamed(double field_bytes) { return field_bytes > 12e6; }

// chunks of the totals' partial sums: of 4096 cells (16 per thread), and at
// most 512, one wave's eight loads per lane in the last sum
constexpr int TOTALS_CELLS = 4096, TOTALS_CHUNKS = 512;
int totals_per_chunk(int n) { return std::max(TOTALS_CELLS, (n - 1) / TOTALS_CHUNKS + 1); }
int totals_chunks(int n) { return (n - 1) / totals_per_chunk(n) + 1; }

Layout layout_of(const int32_t n[3], int precision, bool grav, bool ion)
{
    Layout L;
    size_t N = (size_t)n[0] * n[1] * n[2];
    size_t esz = precision == MHD_FP64 ? 8 : 4;
    size_t nb = (N + NTH - 1) / NTH;
    L.slot = align256(NF * N * esz);
    size_t fbytes = align256(face_values(ion) * N * esz);
    // the face scratch doubles as host staging (MHD_NPRIM or NF FP64 fields)
    size_t stage = align256((size_t)NF * N * 8);
    L.F = 3 * fbytes > stage ? 3 * fbytes : stage;
    // partials: the CFL speed maxima (one per cell-parallel block) and the
    // totals (NF per chunk)
    L.part = align256(std::max(nb, (size_t)NF * totals_chunks((int)N)) * sizeof(double));
    L.misc = 3 * 256;
    // self-gravity: the potential and the FFT tables (the complex scratch of
    // the Poisson solve is the x face scratch, free at that point)
    L.grav = 0;
    if (grav) {
        L.grav = align256(N * esz);
        for (int d = 0; d < 3; d++) L.grav += align256((size_t)n[d] * 2 * esz) + align256(n[d] * 8);
    }
    L.total = 3 * L.slot + L.F + L.part + L.misc + L.grav;
    return L;
}

void box_bind(mhd_box* b, const mhd_params* p, const Layout& L)
{
    b->p = *p;
    b->g = make_geo(p->n[0], p->n[1], p->n[2]);
    b->s = reinterpret_cast<hipStream_t>(p->stream);
    b->prec = p->precision;
    b->esz = p->precision == MHD_FP64 ? 8 : 4;
    b->nblocks = (b->g.n + NTH - 1) / NTH;
    char* w = reinterpret_cast<char*>(p->workspace);
    for (int s = 0; s < 3; s++) {
        b->slot[s] = w;
        w += L.slot;
    }
    size_t fbytes = align256(face_values(p->ionisation != 0) * (size_t)b->g.n * b->esz);
    for (int d = 0; d < 3; d++) b->F[d] = w + d * fbytes;
    w += L.F;
    b->part = reinterpret_cast<double*>(w);
    w += L.part;
    b->flags = reinterpret_cast<uint32_t*>(w);
    b->dt_dev = reinterpret_cast<double*>(w + 256);
    b->tot_dev = reinterpret_cast<double*>(w + 512);
    w += L.misc;
    b->grav = p->grav_G > 0.0;
    b->phi = nullptr;
    for (int d = 0; d < 3; d++) {
        b->tw[d] = nullptr;
        b->sf[d] = nullptr;
    }
    if (b->grav) {
        b->phi = w;
        w += align256((size_t)b->g.n * b->esz);
        for (int d = 0; d < 3; d++) {
            b->tw[d] = w;
            w += align256((size_t)p->n[d] * 2 * b->esz);
            b->sf[d] = reinterpret_cast<double*>(w);
            w += align256((size_t)p->n[d] * 8);
        }
    }
    b->cur[0] = b->cur[1] = b->cur[2] = 0;
    march_segments(b, 1.0);
    b->stream = streamed((double)b->g.n * (double)b->esz);
    b->timing = 0;
    b->nev = 0;
    b->ev_ready = 0;
    for (int c = 0; c < MHD_NKCLASS; c++) {
        b->tms[c] = 0.0;
        b->tcnt[c] = 0;
    }
}

template <typename T>
Fields<T> view(mhd_box* b, int sH, int sM, int sB)
{
    Fields<T> v;
    size_t N = (size_t)b->g.n;
    for (int f = 0; f < NF; f++) {
        int grp = group_of(f);
        int s = grp == GH ? sH : (grp == GM ? sM : sB);
        // without the ionisation network no kernel writes H+: it stays in
        // slot 0, where the state was loaded, whatever slot is current
        if (f == HP && !b->p.ionisation) s = 0;
        v.f[f] = reinterpret_cast<T*>(b->slot[s]) + f * N;
    }
    return v;
}

template <typename T>
CFields<T> cview(const Fields<T>& v)
{
    CFields<T> c;
    for (int f = 0; f < NF; f++) c.f[f] = v.f[f];
    return c;
}

int launch_status() { return hipGetLastError() == hipSuccess ? MHD_OK : MHD_EDEVICE; }

StepArgs step_args(mhd_box* b, double dt, bool dev)
{
    StepArgs a;
    a.gamma = b->p.gamma;
    a.h = 1.0 / (double)b->p.n[0];
    a.dt_val[DT] = dt;
    a.dt_val[DTDX] = dt / a.h;
    a.dt_val[YDX] = b->p.theta * (dt / a.h);
    a.dt_dev = dev ? b->dt_dev : nullptr;
    // the bound is computed from the stored state: FP32 storage moves it by ~1e-7
    a.cfl_tol = b->prec == MHD_FP64 ? 1e-12 : 1e-4;
    a.ion = b->p.ionisation;
    return a;
}

ChemArgs chem_args(mhd_box* b)
{
    ChemArgs c;
    c.on = b->p.chemistry;
    c.cool = b->p.cooling;
    c.ion = b->p.ionisation;
    c.n_unit = b->p.n_unit_cm3;
    c.T_unit = b->p.T_unit_K;
    c.t_unit = b->p.t_unit_s;
    // boxes without chemistry and cooling may have no units
    c.n_inv = c.n_unit > 0.0 ? 1.0 / c.n_unit : 0.0;
    c.e_rate = c.n_unit > 0.0 && c.T_unit > 0.0 ? c.t_unit / (c.n_unit * 1.380649e-16 * c.T_unit) : 0.0;
    return c;
}

const RK rk_coef[3] = { { 0.0, 1.0 }, { 0.75, 0.25 }, { 1.0 / 3.0, 2.0 / 3.0 } };

struct Slots { int h, m, b; };

// ---------------------------------------------------------------- emitters

// event pair around one launch of class cls that holds `parts` of the step's
// kernels (no-op unless timing is on)
struct KTimer {
    mhd_box* b;
    int slot;
    KTimer(mhd_box* box, int cls, int parts) : b(box), slot(-1)
    {
        if (b && b->timing && b->nev < EVCAP) {
            slot = b->nev++;
            b->evcls[slot] = cls;
            b->evparts[slot] = parts;
            (void)hipEventRecord(b->ev[2 * slot], b->s);
        }
    }
    ~KTimer()
    {
        if (slot >= 0) (void)hipEventRecord(b->ev[2 * slot + 1], b->s);
    }
};

int timing_collect(mhd_box* b)
{
    if (!b->timing || b->nev == 0) return MHD_OK;
    if (hipEventSynchronize(b->ev[2 * (b->nev - 1) + 1]) != hipSuccess) return MHD_EDEVICE;
    for (int i = 0; i < b->nev; i++) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, b->ev[2 * i], b->ev[2 * i + 1]) != hipSuccess) return MHD_EDEVICE;
        b->tms[b->evcls[i]] += ms;
        b->tcnt[b->evcls[i]] += b->evparts[i];
    }
    b->nev = 0;
    return MHD_OK;
}

// whether a field of the box is longer than the kernels' 32-bit byte offsets
// reach (more than 2^29 cells in FP64, 2^30 in FP32)
bool wide_fields(const mhd_box* b) { return (uint64_t)b->g.n * b->esz > ((uint64_t)1 << 32); }

// sends each launch of the program straight to the box's stream; O: how the
// kernels reach the fields (Near, Streamed or Far)
template <class O>
struct OneEmit {
    using Access = O;
    mhd_box* b;
    template <class Body>
    void launch(int cls, int blocks, size_t shm, const typename Body::Args& a, int parts = 1)
    {
        if (blocks <= 0) return;
        KTimer t(b, cls, parts);
        if (shm > 65536)
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_one<Body>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
        k_one<Body><<<blocks, Body::NT, shm, b->s>>>(a);
    }
};

// one program position merged over many boxes
struct MultiRec {
    void (*go)(const void* tab, const int* bstart, int nbox, int blocks, size_t shm, hipStream_t s);
    int (*go_persist)(const void* tab, const int* bstart, int nbox, int blocks, size_t shm, hipStream_t s, int ncu,
                      int cap, int* next);
    std::vector<char> args;
    std::vector<int> bstart;
    int total;
    size_t shm;
    size_t off_args, off_bstart;   // offsets in the uploaded table
    size_t off_next;               // the launch's tile counter (uploaded as 0; persistent launches)
};

template <class Body>
void go_many(const void* tab, const int* bstart, int nbox, int blocks, size_t shm, hipStream_t s)
{
    if (shm > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_many<Body>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    k_many<Body><<<blocks, Body::NT, shm, s>>>(reinterpret_cast<const typename Body::Args*>(tab), bstart, nbox);
}

// resident workgroups per CU of k_persist<Body> with shm bytes of dynamic
// LDS (the occupancy query runs once per body and LDS size)
template <class Body>
int persist_per_cu(size_t shm)
{
    static std::mutex mu;
    static std::vector<std::pair<size_t, int>> known;
    std::lock_guard<std::mutex> lk(mu);
    for (const auto& kv : known)
        if (kv.first == shm) return kv.second;
    const void* f = reinterpret_cast<const void*>(&k_persist<Body>);
    if (shm > 65536) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, Body::NT, shm) != hipSuccess || nb < 1) return 0;
    known.push_back(std::make_pair(shm, nb));
    return nb;
}

// claims of tiles per workgroup of a persistent launch: the last claims
// balance the workgroups to within 1 / PERSIST_CLAIMS of their share
constexpr int PERSIST_CLAIMS = 8;

template <class Body>
int go_persist(const void* tab, const int* bstart, int nbox, int blocks, size_t shm, hipStream_t s, int ncu,
               int max_wg, int* next)
{
    if constexpr (!Persists<Body>::v) {
        go_many<Body>(tab, bstart, nbox, blocks, shm, s);
        return MHD_OK;
    } else {
        const int per_cu = persist_per_cu<Body>(shm);
        if (per_cu < 1) return MHD_EDEVICE;
        long cap = (long)per_cu * ncu;
        if (max_wg > 0 && max_wg < cap) cap = max_wg;
        const int grid = blocks < cap ? blocks : (int)cap;
        // about PERSIST_CLAIMS claims per workgroup
        const int chunk = std::max(1, blocks / (grid * PERSIST_CLAIMS));
        k_persist<Body><<<grid, Body::NT, shm, s>>>(reinterpret_cast<const typename Body::Args*>(tab), bstart, nbox,
                                                   blocks, chunk, next);
        return MHD_OK;
    }
}

template <class O>
struct MultiEmit {
    using Access = O;
    std::vector<MultiRec>* recs;
    size_t k;        // program position within the current box
    bool first;      // the first box defines the program
    bool mismatch;
    template <class Body>
    void launch(int, int blocks, size_t shm, const typename Body::Args& a, int = 1)
    {
        if (first) {
            MultiRec r;
            r.go = &go_many<Body>;
            r.go_persist = &go_persist<Body>;
            r.total = 0;
            r.shm = 0;
            r.off_args = r.off_bstart = r.off_next = 0;
            recs->push_back(r);
        }
        if (k >= recs->size() || (*recs)[k].go != &go_many<Body>) {
            mismatch = true;
            return;
        }
        MultiRec& r = (*recs)[k++];
        const char* p = reinterpret_cast<const char*>(&a);
        r.args.insert(r.args.end(), p, p + sizeof(a));
        r.bstart.push_back(r.total);
        r.total += blocks > 0 ? blocks : 0;
        r.shm = shm > r.shm ? shm : r.shm;
    }
};

// ---------------------------------------------------------------- the step program

// longest segment of a marching kernel (longer ones leave the last blocks of
// a large box too uneven: 64 cells cost 1-2% at 256^3)
constexpr int ZMARCH_SEG = 32;

// Segment length of a march over nd cells.  `units` units of work (waves or
// blocks) per segment run on `slots` places (SIMDs or CUs), `occ` at a time on
// each; a further resident unit costs `more` of the time of one alone; starting
// a segment costs `fixed` cells.  A box of few cells wants short segments: a
// march is a serial chain (2 us per face, 3 us per plane of the fused ADV
// update), and 32^3 cells in segments of 32 keep 16 waves busy on 1024 SIMDs
// (1365 us a step; with short ones every launch takes the time of a few
// cells).  A large box wants long ones, whose start is a small part.  The
// parameters are fitted to steps of 32^3 to 256^3 cells at segments of 1 to
// 64; the segments are of even length, so that no launch ends on a short one.
// Only the order of the work depends on the choice, not its results.
int best_segment(int nd, double units, int slots, int occ, double more, double fixed)
{
    int best = 1;
    double cost = 1e300;
    for (int len = nd < ZMARCH_SEG ? nd : ZMARCH_SEG; len >= 1; len--) {
        const int nseg = (nd + len - 1) / len, seg = (nd + nseg - 1) / nseg;
        const double m = std::ceil(units * nseg / slots);
        const double full = std::floor(m / occ), rem = m - full * occ;
        const double c = (full * (1.0 + more * (occ - 1)) + (rem > 0.0 ? 1.0 + more * (rem - 1.0) : 0.0)) * (seg + fixed);
        if (c < cost) {
            cost = c;
            best = seg;
        }
    }
    return best;
}

// tiles of the face-field update: 64 x cells (a wave) by nt / 64 rows for
// blocks of nt threads, narrower for thin boxes
ZTile ztile_of(const Geo& g, int nt, int txmax, int seg)
{
    ZTile z;
    z.tx = g.nx < txmax ? g.nx : txmax;
    z.ty = nt / z.tx;
    z.ntx = (g.nx + z.tx - 1) / z.tx;
    z.nty = (g.ny + z.ty - 1) / z.ty;
    z.seg = seg;
    return z;
}

int ztile_blocks(const Geo& g, const ZTile& z)
{
    return z.ntx * z.nty * ((g.nz + z.seg - 1) / z.seg);
}

// Row segments for blocks of nt threads: the split whose blocks hold the most
// own cells, on a tie the fewer pieces.  A block that is not full costs as much
// as a full one even where whole waves have no cells (they hold registers and
// LDS: FP64 rows of 512 cells as 3 pieces of 171 in three of four waves take
// 96 ps per cell and launch pair of the fused ADV update, as 9 pieces with four
// in a block 82 ps).
RowTile row_tile(int nx, int nt)
{
    RowTile best{};
    double most = -1.0;
    for (int spr = 1; spr <= nx && spr <= 16 + nx / (nt - 6); spr++) {
        RowTile t{};
        t.spr = spr;
        t.tx = (nx + spr - 1) / spr;
        t.w = spr == 1 ? nx : t.tx + 6;
        if (t.w > nt || (long long)t.tx * (spr - 1) >= nx) continue;   // too wide, or an empty last piece
        t.rpb = nt / t.w;
        const double own = (double)nx / spr * t.rpb;
        if (own > most + 1e-9) {
            most = own;
            best = t;
        }
    }
    best.dspr = fast_div(best.spr);
    best.dw = fast_div(best.w);
    return best;
}

// Row segments of the kernels with x rows, in blocks of 256 threads.  FP32
// takes whole rows of up to 512 cells in blocks of 512 where these lose no
// more lanes than the pieces (rows of 512: x-row kernel 791 against 857 us at
// 128 x 512 x 512, fused ADV update 44 against 47 ps per cell and launch pair;
// rows of 367: level).  In FP64 the pieces are faster (rows of 512: 67 against
// 74 and 82 against 90 ps): blocks of 512 leave a CU at two waves per SIMD.
constexpr int ROW_NT = 256;

bool wide_rows(const Geo& g, size_t esz)
{
    if (esz == 8 || g.nx <= ROW_NT || g.nx > 512) return false;
    const RowTile t = row_tile(g.nx, ROW_NT);
    return g.nx / 512.0 >= 0.95 * ((double)g.nx / t.spr * t.rpb / ROW_NT);
}

// segments of the box's marching kernels; the box's share of the launches it
// takes part in is 1 / share (a server's launches cover all boxes in flight)
void march_segments(mhd_box* b, double share)
{
    constexpr int CU = 256, SIMD = 4 * CU;   // MI355X
    const Geo& g = b->g;
    const bool d = b->esz == 8;
    auto waves = [&](double threads) { return share * threads / 64.0; };
    // NONADV faces: two (FP64) or three waves per SIMD; both directions in one
    // launch
    const int occ = d ? 2 : 3;
    const double more = d ? 0.65 : 0.4;
    b->seg_fy = best_segment(g.ny, 2.0 * waves((double)g.nx * g.nz), SIMD, occ, more, d ? 1.5 : 2.5);
    b->seg_fz = best_segment(g.nz, 2.0 * waves((double)g.nx * g.ny), SIMD, occ, more, d ? 1.5 : 2.5);
    b->seg_ay = best_segment(g.ny, waves((double)g.nx * g.nz), SIMD, d ? 2 : 4, d ? 0.65 : 0.35, 2.5);
    // fused ADV update: three (FP64) or four blocks of 256 threads per CU, two
    // of 512; both field groups in one launch (but for FP64 with the network)
    const bool wide = wide_rows(g, b->esz);
    const RowTile rt = row_tile(g.nx, wide ? 512 : ROW_NT);
    const double groups = std::ceil((double)g.ny * rt.spr / rt.rpb);
    b->seg_xz = best_segment(g.nz, (d && b->p.ionisation ? 1.0 : 2.0) * share * groups, CU, wide ? 2 : (d ? 3 : 4), d ? 0.6 : 0.5, 1.0);
    b->seg_b = best_segment(g.nz, waves((double)g.nx * g.ny), SIMD, 4, 0.25, 0.7);
}

// One NONADV substage: y and z faces (marching kernels), the x-row face kernel,
// which also updates m, E and e, and the face-field update.  The primitives are
// formed inside the face kernels from the substage input state.
template <typename T, bool ION, class Emit>
void emit_nonadv_substage_t(mhd_box* b, Emit& e, Slots sin, Slots sS, Slots sout, const StepArgs& a, RK rk,
                            int dbg, bool first)
{
    using O = typename Emit::Access;
    Fields<T> in = view<T>(b, sin.h, sin.m, sin.b);
    Fields<T> S = view<T>(b, sS.h, sS.m, sS.b);
    Fields<T> out = view<T>(b, sout.h, sout.m, sout.b);
    const Geo& g = b->g;
    T* F0 = reinterpret_cast<T*>(b->F[0]);
    T* F1 = reinterpret_cast<T*>(b->F[1]);
    T* F2 = reinterpret_cast<T*>(b->F[2]);
    const T* phi = b->grav ? reinterpret_cast<const T*>(b->phi) : nullptr;
    FaceArgs<T> fa{};
    fa.g = g;
    fa.U = cview(in);
    fa.a = a;
    fa.flags = b->flags;
    fa.dt_cfl = nullptr;
    fa.S = cview(S);
    fa.O = out;
    fa.Fy = F1;
    fa.Fz = F2;
    fa.rk = rk;
    fa.dbg = dbg;
    fa.phi = phi;
    // y and z faces: marching segments
    auto march_blocks = [&](int nd, int no, int seg) {
        const long long threads = (long long)g.nx * no * ((nd + seg - 1) / seg);
        return (int)((threads + NTH - 1) / NTH);
    };
    fa.seg_y = b->seg_fy;
    fa.seg_z = b->seg_fz;
    fa.nby = march_blocks(g.ny, g.nz, fa.seg_y);
    e.template launch<BFaceMarch<T, ION, O>>(MHD_K_NONADV_FACE, fa.nby + march_blocks(g.nz, g.ny, fa.seg_z), 0, fa,
                                           2);
    // x faces; the launch of the first substage checks an explicit dt
    // against the last device CFL bound
    fa.F = F0;
    fa.dt_cfl = first ? b->dt_dev : nullptr;
    const bool wide = wide_rows(g, sizeof(T));
    fa.rt = row_tile(g.nx, wide ? 512 : ROW_NT);
    const int xblocks = (int)(((long long)g.ny * g.nz * fa.rt.spr + fa.rt.rpb - 1) / fa.rt.rpb);
    if constexpr (sizeof(T) == 4) {
        if (wide)
            e.template launch<BFaceXRows<T, 512, ION, O>>(MHD_K_NONADV_FACE, xblocks, 512 * XROW_SLOTS * sizeof(T), fa);
    }
    if (!wide)
        e.template launch<BFaceXRows<T, ROW_NT, ION, O>>(MHD_K_NONADV_FACE, xblocks, ROW_NT * XROW_SLOTS * sizeof(T), fa);
    FieldUpdateArgs<T> ua;
    ua.g = g;
    ua.U = cview(in);
    ua.S = cview(S);
    ua.O = out;
    ua.Fx = F0;
    ua.Fy = F1;
    ua.Fz = F2;
    ua.a = a;
    ua.rk = rk;
    ua.dbg = dbg;
    ua.zt = ztile_of(g, UPD_NT, UPD_TX, b->seg_b);
    e.template launch<BFieldUpdate<T, O>>(MHD_K_NONADV_UPDATE, ztile_blocks(g, ua.zt), 0, ua);
}

template <typename T, class Emit>
void emit_nonadv_substage(mhd_box* b, Emit& e, Slots sin, Slots sS, Slots sout, const StepArgs& a, RK rk, int dbg,
                          bool first)
{
    if (b->p.ionisation)
        emit_nonadv_substage_t<T, true>(b, e, sin, sS, sout, a, rk, dbg, first);
    else
        emit_nonadv_substage_t<T, false>(b, e, sin, sS, sout, a, rk, dbg, first);
}

// ADV faces along y, marched along y
template <typename T, int NQ, class Emit>
void emit_adv_face(mhd_box* b, Emit& e, const Fields<T>& in, const StepArgs& a)
{
    using O = typename Emit::Access;
    typename BAdvFaceMarchY<T, NQ, O>::Args ma;
    ma.g = b->g;
    ma.U = cview(in);
    ma.a = a;
    ma.F = reinterpret_cast<T*>(b->F[1]);
    ma.seg = b->seg_ay;
    long long threads = (long long)b->g.nx * b->g.nz * ((b->g.ny + ma.seg - 1) / ma.seg);
    e.template launch<BAdvFaceMarchY<T, NQ, O>>(MHD_K_ADV_FACE, (int)((threads + NTH - 1) / NTH), 0, ma);
}

// the fused ADV update with blocks of NT threads, one launch for both field
// groups where their registers allow (dynamic LDS: 2 x (NV + 2 NQ) x NT values)
template <typename T, int NT, class Emit>
void emit_adv_xz(Emit& e, const AdvXZArgs<T>& xa, bool ion)
{
    using O = typename Emit::Access;
    auto shm = [](int nv, int nq) { return (size_t)2 * (nv + 2 * nq) * NT * sizeof(T); };
    const int both = 2 * xa.tiles;
    if (!ion) {
        e.template launch<BAdvXZPair<T, 3, NT, O>>(MHD_K_ADV_UPDATE, both, shm(4, 4), xa, 2);
    } else if constexpr (sizeof(T) == 4) {
        e.template launch<BAdvXZPair<T, 4, NT, O>>(MHD_K_ADV_UPDATE, both, shm(6, 4), xa, 2);
    } else {
        e.template launch<BAdvXZUpdate<T, 0, 4, NT, O>>(MHD_K_ADV_UPDATE, xa.tiles, shm(4, 4), xa);   // rho, m
        e.template launch<BAdvXZUpdate<T, 4, 4, NT, O>>(MHD_K_ADV_UPDATE, xa.tiles, shm(6, 4), xa);   // E, e, h2, hp
    }
}

// One ADV substage: y faces marched along y, then the update with its x and z
// faces
template <typename T, class Emit>
void emit_adv_substage(mhd_box* b, Emit& e, Slots sin, Slots sS, Slots sout, const StepArgs& a, RK rk, int dbg)
{
    Fields<T> in = view<T>(b, sin.h, sin.m, sin.b);
    Fields<T> S = view<T>(b, sS.h, sS.m, sS.b);
    Fields<T> out = view<T>(b, sout.h, sout.m, sout.b);
    const bool ion = b->p.ionisation != 0;
    if (ion) emit_adv_face<T, 8>(b, e, in, a);
    else emit_adv_face<T, 7>(b, e, in, a);
    AdvXZArgs<T> xa;
    xa.g = b->g;
    xa.U = cview(in);
    xa.S = cview(S);
    xa.O = out;
    xa.Fy = reinterpret_cast<T*>(b->F[1]);
    xa.a = a;
    xa.rk = rk;
    xa.dbg = dbg;
    const bool wide = wide_rows(b->g, sizeof(T));
    xa.rt = row_tile(b->g.nx, wide ? 512 : ROW_NT);
    xa.nrg = (int)(((long long)b->g.ny * xa.rt.spr + xa.rt.rpb - 1) / xa.rt.rpb);
    xa.seg = b->seg_xz;
    xa.tiles = xa.nrg * ((b->g.nz + xa.seg - 1) / xa.seg);
    if constexpr (sizeof(T) == 4) {
        if (wide) emit_adv_xz<T, 512>(e, xa, ion);
    }
    if (!wide) emit_adv_xz<T, ROW_NT>(e, xa, ion);
}

// NONADV stage: the M and B groups each rotate through their three slots
// (stage start S, then A, B, A); H is read from its current slot.
template <typename T, class Emit>
void emit_nonadv_stage(mhd_box* b, Emit& e, const StepArgs& a, bool first)
{
    int h = b->cur[GH], Sm = b->cur[GM], Sb = b->cur[GB];
    Slots S0 = { h, Sm, Sb };
    Slots A = { h, (Sm + 1) % 3, (Sb + 1) % 3 };
    Slots B2 = { h, (Sm + 2) % 3, (Sb + 2) % 3 };
    emit_nonadv_substage<T>(b, e, S0, S0, A, a, rk_coef[0], 0, first);
    emit_nonadv_substage<T>(b, e, A, S0, B2, a, rk_coef[1], 0, false);
    emit_nonadv_substage<T>(b, e, B2, S0, A, a, rk_coef[2], 0, false);
    b->cur[GM] = A.m;
    b->cur[GB] = A.b;
}

// ADV stage: the H and M groups rotate; B is read from its current slot
template <typename T, class Emit>
void emit_adv_stage(mhd_box* b, Emit& e, const StepArgs& a)
{
    int Sh = b->cur[GH], Sm = b->cur[GM], bb = b->cur[GB];
    Slots S0 = { Sh, Sm, bb };
    Slots A = { (Sh + 1) % 3, (Sm + 1) % 3, bb };
    Slots B2 = { (Sh + 2) % 3, (Sm + 2) % 3, bb };
    emit_adv_substage<T>(b, e, S0, S0, A, a, rk_coef[0], 0);
    emit_adv_substage<T>(b, e, A, S0, B2, a, rk_coef[1], 0);
    emit_adv_substage<T>(b, e, B2, S0, A, a, rk_coef[2], 0);
    b->cur[GH] = A.h;
    b->cur[GM] = A.m;
}

// dt from the per-block CFL speed maxima in b->part
template <class Emit>
void emit_reduce_dt(mhd_box* b, Emit& e, int nparts)
{
    BReduceDt::Args ra;
    ra.part = b->part;
    ra.nparts = nparts;
    ra.cflh = b->p.cfl * (1.0 / (double)b->p.n[0]);
    ra.h = 1.0 / (double)b->p.n[0];
    ra.theta = b->p.theta;
    ra.dt = b->dt_dev;
    e.template launch<BReduceDt>(MHD_K_REDUCE, 1, 0, ra);
}

template <typename T, class Emit>
void emit_tail(mhd_box* b, Emit& e, const StepArgs& a, int mode)
{
    using O = typename Emit::Access;
    typename BTail<T, O>::Args ta;
    ta.g = b->g;
    ta.U = view<T>(b, b->cur[GH], b->cur[GM], b->cur[GB]);
    ta.a = a;
    ta.ch = chem_args(b);
    ta.mode = mode;
    ta.part = b->part;
    ta.flags = b->flags;
    e.template launch<BTail<T, O>>(MHD_K_TAIL, b->nblocks, 0, ta);
    emit_reduce_dt(b, e, b->nblocks);
}

int ilog2(int n)
{
    int l = 0;
    while ((1 << l) < n) l++;
    return l;
}

// Poisson stage (Sec. 2.9) on the current density: x forward, y forward,
// z forward + Green's function + z inverse, y inverse, x inverse
template <typename T, class Emit>
void emit_poisson(mhd_box* b, Emit& e)
{
    const Geo& g = b->g;
    FftArgs<T> fa;
    fa.g = g;
    fa.rho = reinterpret_cast<const T*>(b->slot[b->cur[GH]]) + (size_t)RHO * g.n;
    fa.Z = reinterpret_cast<Cx<T>*>(b->F[0]);
    fa.phi = reinterpret_cast<T*>(b->phi);
    for (int d = 0; d < 3; d++) {
        fa.tw[d] = reinterpret_cast<const Cx<T>*>(b->tw[d]);
        fa.sf[d] = b->sf[d];
        fa.logn[d] = ilog2(b->p.n[d]);
    }
    const double h = 1.0 / (double)b->p.n[0];
    fa.gscale = -(2.0 / 3.0) * M_PI * b->p.grav_G * h * h / (double)g.n;
    fa.lpb = g.nx >= FFT_X_VALUES ? 1 : FFT_X_VALUES / g.nx;
    const int lines = g.ny * g.nz;
    const int xb = (lines + fa.lpb - 1) / fa.lpb;
    const size_t xshm = (size_t)fa.lpb * g.nx * sizeof(Cx<T>);
    e.template launch<BFftX<T, 0>>(MHD_K_POISSON, xb, xshm, fa);
    // y and z passes: tx columns of a line set, tx x (n + 1) complex in LDS
    // (powers of two, like the axes)
    auto pass = [&](int n) {
        const int t = std::min(FFT_YZ_VALUES / n, g.nx);
        fa.logt = ilog2(t);
        return t;
    };
    int tx = pass(g.ny);
    e.template launch<BFftYZ<T, 1, 0>>(MHD_K_POISSON, (g.nx / tx) * g.nz,
                                       (size_t)tx * (g.ny + 1) * sizeof(Cx<T>), fa);
    tx = pass(g.nz);
    e.template launch<BFftYZ<T, 2, 2>>(MHD_K_POISSON, (g.nx / tx) * g.ny,
                                       (size_t)tx * (g.nz + 1) * sizeof(Cx<T>), fa);
    tx = pass(g.ny);
    e.template launch<BFftYZ<T, 1, 1>>(MHD_K_POISSON, (g.nx / tx) * g.nz,
                                       (size_t)tx * (g.ny + 1) * sizeof(Cx<T>), fa);
    e.template launch<BFftX<T, 1>>(MHD_K_POISSON, xb, xshm, fa);
}

// host-built FFT tables of a self-gravity box, uploaded on the box's stream;
// the caller synchronises before `host` goes out of scope
template <typename T>
int upload_grav_tables(mhd_box* b, std::vector<double>& host)
{
    if (!b->grav) return MHD_OK;
    for (int d = 0; d < 3; d++) {
        const int n = b->p.n[d];
        std::vector<T> tw((size_t)n * 2, T(0));
        for (int m = 0; m < n; m++) {
            const double t = 2.0 * M_PI * (double)m / (double)n;
            tw[2 * m] = (T)std::cos(t);
            tw[2 * m + 1] = (T)(-std::sin(t));
        }
        const size_t off = host.size();
        host.resize(off + (tw.size() * sizeof(T) + 7) / 8 + n);
        std::memcpy(host.data() + off, tw.data(), tw.size() * sizeof(T));
        double* sfh = host.data() + off + (tw.size() * sizeof(T) + 7) / 8;
        for (int m = 0; m < n; m++) {
            const double s = std::sin(M_PI * (double)m / (double)n);
            sfh[m] = (3.0 - 2.0 * s * s) / 3.0;
        }
    }
    size_t off = 0;
    for (int d = 0; d < 3; d++) {
        const int n = b->p.n[d];
        const size_t twb = (size_t)n * 2 * sizeof(T);
        if (hipMemcpyAsync(b->tw[d], host.data() + off, twb, hipMemcpyHostToDevice, b->s) != hipSuccess)
            return MHD_EDEVICE;
        off += (twb + 7) / 8;
        if (hipMemcpyAsync(b->sf[d], host.data() + off, (size_t)n * 8, hipMemcpyHostToDevice, b->s) !=
            hipSuccess)
            return MHD_EDEVICE;
        off += n;
    }
    return MHD_OK;
}

template <typename T, class Emit>
void emit_step(mhd_box* b, Emit& e, const StepArgs& a)
{
    if (b->grav) emit_poisson<T>(b, e);
    emit_nonadv_stage<T>(b, e, a, true);
    emit_adv_stage<T>(b, e, a);
    emit_tail<T>(b, e, a, 1);
}

// ---------------------------------------------------------------- single-box operations

// f(e) with the box's emitter
template <class F>
void with_emit(mhd_box* b, F&& f)
{
    if (wide_fields(b)) {
        OneEmit<Far> e{ b };
        f(e);
    } else if (b->stream) {
        OneEmit<Streamed> e{ b };
        f(e);
    } else {
        OneEmit<Near> e{ b };
        f(e);
    }
}

template <typename T>
int full_step(mhd_box* b, double dt, bool dev)
{
    StepArgs a = step_args(b, dt, dev);
    with_emit(b, [&](auto& e) { emit_step<T>(b, e, a); });
    int st = launch_status();
    if (st) return st;
    // the event ring is read (a wait on its last event) only once half of it
    // is used, so timed steps stay asynchronous
    return b->nev >= EVCAP / 2 ? timing_collect(b) : MHD_OK;
}

int flags_status(uint32_t fl)
{
    if (fl & 1u) return MHD_ENONPHYS;
    if (fl & 2u) return MHD_ECFL;
    return MHD_OK;
}

int sync_and_flags(mhd_box* b)
{
    uint32_t fl = 0;
    if (hipMemcpyAsync(&fl, b->flags, sizeof(fl), hipMemcpyDeviceToHost, b->s) != hipSuccess) return MHD_EDEVICE;
    if (hipStreamSynchronize(b->s) != hipSuccess) return MHD_EDEVICE;
    return flags_status(fl);
}

// ---------------------------------------------------------------- host copies

// threads that copy `bytes` of host memory beside the caller's (0: too little
// to be worth starting one): fresh pages of the caller's are
// zeroed by the kernel as they are first written, at about 20 GB/s per thread
// with large pages and a fifth of that without
int copy_threads(size_t bytes)
{
    const size_t most = std::min<size_t>(8, std::max(1u, std::thread::hardware_concurrency()));
    const size_t n = std::min<size_t>(most, bytes / ((size_t)2 << 20));
    return n > 1 ? (int)n : 0;
}

// Runs work(t, nt) on nt threads beside the caller's own lead(nt), nt at most
// `threads` (fewer where the system gives no more; none: lead(0) does the work).
template <class Lead, class Work>
int with_threads(int threads, Lead&& lead, Work&& work)
{
    std::vector<std::thread> pool;
    std::atomic<int> go{ -1 };
    try {
        pool.reserve(threads);
        for (int t = 0; t < threads; t++)
            pool.emplace_back([&, t] {
                int nt;
                while ((nt = go.load(std::memory_order_acquire)) < 0) std::this_thread::yield();
                work(t, nt);
            });
    } catch (...) {   // no further thread: go on with those there are
    }
    const int nt = (int)pool.size();
    go.store(nt, std::memory_order_release);
    const int st = lead(nt);
    for (std::thread& t : pool) t.join();
    return st;
}

// memcpy of host memory by several threads
void host_copy(void* dst, const void* src, size_t bytes)
{
    auto part = [&](int t, int nt) {
        const size_t a = bytes / nt * t, e = t + 1 == nt ? bytes : bytes / nt * (t + 1);
        memcpy(static_cast<char*>(dst) + a, static_cast<const char*>(src) + a, e - a);
    };
    with_threads(copy_threads(bytes),
                 [&](int nt) {
                     if (nt == 0) part(0, 1);
                     return MHD_OK;
                 },
                 part);
}

// Makes the ring ready for a state of this many bytes on the stream.  False,
// for the runtime's own copy, without the memory or the events for it; on a
// stream that is being captured, where copies are only recorded (the runtime's
// refuses); and on a stream of another device than the events'.
bool ring_ready(HostRing& r, size_t bytes, hipStream_t s)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return false;
    }
    const size_t want = std::min(RING_SLOT_MAX, align256((bytes + RING_SLOTS - 1) / RING_SLOTS));
    if (r.mem && r.slot < want) {   // a server's ring, sized for a smaller box
        (void)hipHostFree(r.mem);
        r.mem = nullptr;
    }
    if (!r.mem) {
        if (hipHostMalloc(reinterpret_cast<void**>(&r.mem), RING_SLOTS * want + 256, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            r.mem = nullptr;
            return false;
        }
        r.slot = want;
    }
    while (r.nev < RING_SLOTS) {
        if (hipEventCreateWithFlags(&r.ev[r.nev], hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        r.nev++;
    }
    if (hipEventRecord(r.ev[0], s) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return true;
}

void ring_release(HostRing& r)
{
    for (int i = 0; i < r.nev; i++) (void)hipEventDestroy(r.ev[i]);
    if (r.mem) (void)hipHostFree(r.mem);
    r.mem = nullptr;
    r.nev = 0;
}

// Device ranges of values to consecutive FP64 values of pageable host memory,
// and the fault flags.  The values pass through the ring's pinned slots in the
// order of the ranges: this thread keeps the copies to the slots queued and
// announces each that has arrived, the others copy (and widen) its slices to
// the caller's memory.  Before the first one arrives, while steps still run,
// they write a byte to every page of their slices, so that the pages are there.
// (Straight into fresh pageable memory the runtime copies at 10 GB/s; a 256^3
// FP64 state, 1.48 GB, takes 150 ms that way.  FP32 values cross the link as
// they are and are widened here, exactly.)
struct Range {
    const void* dev;
    size_t n;
};

template <typename T>
int copy_out(hipStream_t s, HostRing& ring, const Range* ranges, int nranges, double* host, const uint32_t* flags_dev,
             uint32_t* flags)
{
    const size_t most = ring.slot / sizeof(T);   // values per chunk
    struct Chunk {
        const T* dev;
        double* dst;
        size_t n;
    };
    std::vector<Chunk> ch;
    size_t total = 0;
    for (int r = 0; r < nranges; r++) {
        for (size_t o = 0; o < ranges[r].n; o += most)
            ch.push_back({ static_cast<const T*>(ranges[r].dev) + o, host + total + o,
                           std::min(most, ranges[r].n - o) });
        total += ranges[r].n;
    }
    const int nch = (int)ch.size();
    std::atomic<int> arrived{ 0 };            // chunks in the slots (past nch: give up)
    std::atomic<int> taken[RING_SLOTS] = {};  // slices copied out of each slot
    uint32_t* fl = reinterpret_cast<uint32_t*>(ring.mem + RING_SLOTS * ring.slot);
    auto slot = [&](int k) { return reinterpret_cast<T*>(ring.mem + (size_t)(k % RING_SLOTS) * ring.slot); };
    auto take = [&](int k, int t, int nt) {
        const Chunk& c = ch[k];
        const size_t a = c.n / nt * t, e = t + 1 == nt ? c.n : c.n / nt * (t + 1);
        const T* src = slot(k);
        if constexpr (sizeof(T) == sizeof(double)) {
            memcpy(c.dst + a, src + a, (e - a) * sizeof(double));
        } else {
            for (size_t i = a; i < e; i++) c.dst[i] = (double)src[i];
        }
    };
    auto work = [&](int t, int nt) {
        for (int k = 0; k < nch && arrived.load(std::memory_order_relaxed) == 0; k++) {
            const size_t a = ch[k].n / nt * t, e = t + 1 == nt ? ch[k].n : ch[k].n / nt * (t + 1);
            for (size_t i = a; i < e; i += 4096 / sizeof(double)) *(volatile char*)(ch[k].dst + i) = 0;
        }
        for (int k = 0; k < nch; k++) {
            int n;
            for (int spin = 0; (n = arrived.load(std::memory_order_acquire)) <= k; spin++) {
                if (spin < 1000) std::this_thread::yield();
                else std::this_thread::sleep_for(std::chrono::microseconds(20));
            }
            if (n > nch) return;
            take(k, t, nt);
            taken[k % RING_SLOTS].fetch_add(1, std::memory_order_release);
        }
    };
    // a slot is filled again LAG chunks after the announcement of the chunk it
    // held, so that a slow thread does not hold up the next announcement
    constexpr int LAG = 2;
    auto lead = [&](int nt) {
        int st = MHD_OK;
        auto issue = [&](int k) {
            if (k >= RING_SLOTS && nt > 0)
                while (taken[k % RING_SLOTS].load(std::memory_order_acquire) < nt * (k / RING_SLOTS))
                    std::this_thread::yield();
            if (hipMemcpyAsync(slot(k), ch[k].dev, ch[k].n * sizeof(T), hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipEventRecord(ring.ev[k % RING_SLOTS], s) != hipSuccess)
                st = MHD_EDEVICE;
        };
        if (hipMemcpyAsync(fl, flags_dev, sizeof(uint32_t), hipMemcpyDeviceToHost, s) != hipSuccess) st = MHD_EDEVICE;
        int issued = 0;
        for (; st == MHD_OK && issued < nch && issued < RING_SLOTS - LAG; issued++) issue(issued);
        for (int k = 0; st == MHD_OK && k < nch; k++) {
            if (hipEventSynchronize(ring.ev[k % RING_SLOTS]) != hipSuccess) {
                st = MHD_EDEVICE;
                break;
            }
            if (nt == 0) take(k, 0, 1);
            arrived.store(k + 1, std::memory_order_release);
            if (issued < nch) issue(issued++);
        }
        if (st != MHD_OK) arrived.store(nch + 1, std::memory_order_release);
        return st;
    };
    const int st = with_threads(copy_threads(total * sizeof(double)), lead, work);
    if (st != MHD_OK) return st;
    *flags = *fl;
    return MHD_OK;
}

template <typename T>
int load_f64(mhd_box* b, const double* host, bool prim, bool wait = true)
{
    size_t N = (size_t)b->g.n;
    double* stage = reinterpret_cast<double*>(b->F[0]);
    size_t nf = prim ? MHD_NPRIM : NF;
    if (hipMemcpyAsync(stage, host, nf * N * sizeof(double), hipMemcpyHostToDevice, b->s) != hipSuccess)
        return MHD_EDEVICE;
    std::vector<double> tables;
    int tst = upload_grav_tables<T>(b, tables);
    if (tst) return tst;
    b->cur[GH] = b->cur[GM] = b->cur[GB] = 0;
    Fields<T> u = view<T>(b, 0, 0, 0);
    int saved = b->timing;
    b->timing = 0;
    with_emit(b, [&](auto& e) {
        if (prim) {
            typename BInit<T>::Args ia;
            ia.g = b->g;
            ia.Wp = stage;
            ia.U = u;
            ia.gamma = b->p.gamma;
            ia.ion = b->p.ionisation;
            e.template launch<BInit<T>>(MHD_K_SETUP, b->nblocks, 0, ia);
        } else {
            typename BFromF64<T>::Args ia;
            ia.g = b->g;
            ia.src = stage;
            ia.U = u;
            e.template launch<BFromF64<T>>(MHD_K_SETUP, b->nblocks, 0, ia);
        }
        BClearFlags::Args ca;
        ca.flags = b->flags;
        e.template launch<BClearFlags>(0, 1, 0, ca);
        StepArgs a = step_args(b, 0.0, false);
        emit_tail<T>(b, e, a, 0);
    });
    b->timing = saved;
    int st = launch_status();
    if (st) return st;
    if (wait && hipStreamSynchronize(b->s) != hipSuccess) return MHD_EDEVICE;
    return MHD_OK;
}

// whether the runtime knows this memory: pinned host memory, to which it copies
// at the rate of the link, and managed or device memory, which host threads may
// not be able to write
bool runtime_memory(const void* host)
{
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, host) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return at.type != hipMemoryTypeUnregistered;
}

// states below this many FP64 bytes leave in one copy of the runtime's (32^3,
// 2.9 MB: 0.21 ms, through the ring 0.23 ms and 1 ms more at its first use)
constexpr size_t RING_MIN = (size_t)8 << 20;

// the current state to host FP64 (the groups H, M, B in host field order)
template <typename T>
int get_f64(mhd_box* b, HostRing& ring, double* host)
{
    const size_t N = (size_t)b->g.n;
    const Fields<T> u = view<T>(b, b->cur[GH], b->cur[GM], b->cur[GB]);
    if (NF * N * sizeof(double) < RING_MIN || runtime_memory(host) || !ring_ready(ring, NF * N * sizeof(T), b->s)) {
        typename BToF64<T>::Args ta;
        ta.g = b->g;
        ta.U = cview(u);
        ta.dst = reinterpret_cast<double*>(b->F[0]);
        k_one<BToF64<T>><<<b->nblocks, NTH, 0, b->s>>>(ta);
        if (launch_status()) return MHD_EDEVICE;
        if (hipMemcpyAsync(host, ta.dst, NF * N * sizeof(double), hipMemcpyDeviceToHost, b->s) != hipSuccess)
            return MHD_EDEVICE;
        return sync_and_flags(b);
    }
    static_assert(RHO == 0 && MX == 1 && EI == 5 && BX == 6 && BZ == 8 && H2 == 9 && HP == 10 && NF == 11,
                  "groups of the host field order");
    const Range r[5] = { { u.f[RHO], N }, { u.f[MX], 5 * N }, { u.f[BX], 3 * N }, { u.f[H2], N }, { u.f[HP], N } };
    uint32_t fl = 0;
    int st;
    try {
        st = copy_out<T>(b->s, ring, r, 5, host, b->flags, &fl);
    } catch (const std::bad_alloc&) {
        return MHD_ENOMEM;
    }
    return st ? st : flags_status(fl);
}

template <typename T>
int totals_run(const CFields<T>& u, int n, hipStream_t s, double* part, double* out)
{
    typename BTotalsPartial<T>::Args pa;
    pa.n = n;
    pa.per = totals_per_chunk(n);
    pa.chunks = totals_chunks(n);
    pa.U = u;
    pa.part = part;
    k_one<BTotalsPartial<T>><<<NF * pa.chunks, NTH, 0, s>>>(pa);
    BTotalsFinal::Args fa;
    fa.part = part;
    fa.chunks = pa.chunks;
    fa.out = out;
    k_one<BTotalsFinal><<<1, BTotalsFinal::NT, 0, s>>>(fa);
    return launch_status();
}

template <typename T>
int totals_launch(mhd_box* b)
{
    return totals_run<T>(cview(view<T>(b, b->cur[GH], b->cur[GM], b->cur[GB])), b->g.n, b->s, b->part, b->tot_dev);
}

template <typename T>
int totals(mhd_box* b, double* out)
{
    if (totals_launch<T>(b)) return MHD_EDEVICE;
    if (hipMemcpyAsync(out, b->tot_dev, NF * sizeof(double), hipMemcpyDeviceToHost, b->s) != hipSuccess)
        return MHD_EDEVICE;
    return sync_and_flags(b);
}

template <typename T>
int debug_stage(mhd_box* b, int stage, double dt)
{
    StepArgs a = step_args(b, dt, false);
    int st = MHD_OK;
    with_emit(b, [&](auto& e) {
        if (b->grav && (stage == MHD_STAGE_NONADV || stage == MHD_STAGE_NONADV_RHS)) emit_poisson<T>(b, e);
        switch (stage) {
        case MHD_STAGE_NONADV: emit_nonadv_stage<T>(b, e, a, false); break;
        case MHD_STAGE_ADV: emit_adv_stage<T>(b, e, a); break;
        case MHD_STAGE_TAIL: emit_tail<T>(b, e, a, 1); break;
        case MHD_STAGE_NONADV_RHS:
        case MHD_STAGE_ADV_RHS: {
            // tau R(U) of one substage into all ten fields of a free slot; needs
            // the three groups in one slot (true right after mhd_set_state)
            int S = b->cur[GM];
            if (b->cur[GH] != S || b->cur[GB] != S) {
                st = MHD_EINVAL;
                return;
            }
            int O = (S + 1) % 3;
            Slots s0 = { S, S, S }, so = { O, O, O };
            if (stage == MHD_STAGE_NONADV_RHS)
                emit_nonadv_substage<T>(b, e, s0, s0, so, a, rk_coef[0], 1, false);
            else
                emit_adv_substage<T>(b, e, s0, s0, so, a, rk_coef[0], 1);
            b->cur[GH] = b->cur[GM] = b->cur[GB] = O;
            break;
        }
        default: st = MHD_EINVAL;
        }
    });
    return st ? st : launch_status();
}

double now_s()
{
    using namespace std::chrono;
    return duration<double>(steady_clock::now().time_since_epoch()).count();
}

}  // namespace

// ---------------------------------------------------------------- server

// FP64 values of a request or a result in host memory, not initialised
struct HostState {
    std::unique_ptr<double[]> v;
    size_t n = 0;
    bool resize(size_t count)
    {
        v.reset(new (std::nothrow) double[count]);
        n = v ? count : 0;
        return n == count;
    }
};

struct mhd_server {
    mhd_server_params p;
    hipStream_t s;
    char* dtab;                // device launch tables (start of the workspace)
    char* htab;                // pinned host copy of the tables
    char* pool;                // the rest of the workspace: box allocations
    size_t pool_bytes;
    std::vector<std::pair<size_t, size_t>> freel;   // (offset, size), sorted by offset
    size_t used, peak;
    struct Pending {
        uint64_t id;
        mhd_request r;
        HostState prim;                 // copied state, or
        const double* src = nullptr;    // the caller's state, borrowed
        double t_submit;
    };
    struct Active {
        uint64_t id;
        mhd_box* box;
        size_t off, bytes;
        int steps, done, keep;
        double t_submit, t_admit;
    };
    std::deque<Pending> pending;
    std::vector<Active> active;
    std::deque<mhd_completion> done;
    std::unordered_map<uint64_t, HostState> results;
    HostRing ring;
    uint64_t next_id;
    double t0;
    std::vector<MultiRec> recs;
    // pipelined rounds: a call launches its round and then waits for the one
    // before.  A box is in exactly one of: active, retiring (by the half of the
    // round that finishes it; its totals and flags are on the way to the pinned
    // slot of its place in the list), finished (round over, totals and flags at
    // hand, not reported yet: the report needs host memory and is tried again by
    // the next call if there is none)
    struct Finished {
        Active a;
        double totals[NF];
        uint32_t flags;
    };
    std::list<Finished> retiring[2], finished;
    hipEvent_t ev[2];
    int ev_ready;
    int64_t rounds;        // rounds launched
    int ncu;               // compute units of the server's device (persistent launches)
    bool prev_launched;    // the previous call launched a round (event ev[(rounds - 1) & 1])
};

namespace {

constexpr size_t SERVER_TAB_BYTES = (size_t)32 << 20;   // launch tables of one round
constexpr int SERVER_MAX_SLOTS = 1024;
// pinned return slot of a finished box: NF totals and the fault flags
constexpr size_t SERVER_RET_BYTES = (NF + 1) * sizeof(double);
// pinned host area: two table halves (consecutive rounds alternate) and two
// sets of return slots
constexpr size_t SERVER_HOST_BYTES = 2 * SERVER_TAB_BYTES + 2 * SERVER_MAX_SLOTS * SERVER_RET_BYTES;
constexpr int SERVER_MAX_NX = 256;

bool pool_alloc(mhd_server* sv, size_t bytes, size_t* off)
{
    bytes = align256(bytes);
    for (size_t i = 0; i < sv->freel.size(); i++) {
        if (sv->freel[i].second >= bytes) {
            *off = sv->freel[i].first;
            sv->freel[i].first += bytes;
            sv->freel[i].second -= bytes;
            if (sv->freel[i].second == 0) sv->freel.erase(sv->freel.begin() + i);
            sv->used += bytes;
            if (sv->used > sv->peak) sv->peak = sv->used;
            return true;
        }
    }
    return false;
}

void pool_free(mhd_server* sv, size_t off, size_t bytes)
{
    bytes = align256(bytes);
    sv->used -= bytes;
    size_t i = 0;
    while (i < sv->freel.size() && sv->freel[i].first < off) i++;
    sv->freel.insert(sv->freel.begin() + i, std::make_pair(off, bytes));
    if (i + 1 < sv->freel.size() && sv->freel[i].first + sv->freel[i].second == sv->freel[i + 1].first) {
        sv->freel[i].second += sv->freel[i + 1].second;
        sv->freel.erase(sv->freel.begin() + i + 1);
    }
    if (i > 0 && sv->freel[i - 1].first + sv->freel[i - 1].second == sv->freel[i].first) {
        sv->freel[i - 1].second += sv->freel[i].second;
        sv->freel.erase(sv->freel.begin() + i);
    }
}

mhd_params box_params(const mhd_server* sv, const int32_t n[3], void* ws, size_t bytes)
{
    mhd_params bp;
    bp.n[0] = n[0];
    bp.n[1] = n[1];
    bp.n[2] = n[2];
    bp.gamma = sv->p.gamma;
    bp.cfl = sv->p.cfl;
    bp.precision = sv->p.precision;
    bp.theta = sv->p.theta;
    bp.chemistry = sv->p.chemistry;
    bp.cooling = sv->p.cooling;
    bp.grav_G = 0.0;   // served boxes run without self-gravity
    bp.ionisation = 0; // and without the ionisation network
    bp.n_unit_cm3 = sv->p.n_unit_cm3;
    bp.T_unit_K = sv->p.T_unit_K;
    bp.t_unit_s = sv->p.t_unit_s;
    bp.stream = sv->p.stream;
    bp.workspace = ws;
    bp.workspace_bytes = bytes;
    return bp;
}

int server_admit(mhd_server* sv)
{
    while (!sv->pending.empty() && (int)sv->active.size() < sv->p.max_slots) {
        mhd_server::Pending& q = sv->pending.front();
        Layout L = layout_of(q.r.n, sv->p.precision, false, false);
        size_t off;
        if (!pool_alloc(sv, L.total, &off)) break;   // first come, first served: wait for memory
        mhd_box* b = new (std::nothrow) mhd_box;
        if (!b) {
            pool_free(sv, off, L.total);
            return MHD_ENOMEM;
        }
        mhd_params bp = box_params(sv, q.r.n, sv->pool + off, L.total);
        box_bind(b, &bp, L);
        // a copied state is freed below, so its upload completes first; a
        // borrowed one stays valid until the completion is polled
        const double* src = q.src ? q.src : q.prim.v.get();
        const bool wait = q.src == nullptr;
        int st = sv->p.precision == MHD_FP64 ? load_f64<double>(b, src, true, wait)
                                             : load_f64<float>(b, src, true, wait);
        if (st) {
            delete b;
            pool_free(sv, off, L.total);
            return st;
        }
        mhd_server::Active a;
        a.id = q.id;
        a.box = b;
        a.off = off;
        a.bytes = L.total;
        a.steps = q.r.steps;
        a.done = 0;
        a.keep = q.r.keep_state;
        a.t_submit = q.t_submit;
        a.t_admit = now_s() - sv->t0;
        sv->active.push_back(a);
        sv->pending.pop_front();
    }
    return MHD_OK;
}

// one step of every active box, merged into one launch per program position
template <typename T, class O>
int server_step(mhd_server* sv, int half)
{
    sv->recs.clear();
    MultiEmit<O> e{ &sv->recs, 0, true, false };
    double cells = 0.0;
    for (const mhd_server::Active& a : sv->active) cells += (double)a.box->g.n;
    for (size_t i = 0; i < sv->active.size(); i++) {
        mhd_box* b = sv->active[i].box;
        e.k = 0;
        e.first = i == 0;
        march_segments(b, cells / (double)b->g.n);
        StepArgs a = step_args(b, 0.0, true);
        emit_step<T>(b, e, a);
        if (e.mismatch || e.k != sv->recs.size()) return MHD_EINVAL;
    }
    // pack the tables into this round's half and upload them once
    size_t off = 0;
    for (MultiRec& r : sv->recs) {
        off = align256(off);
        r.off_args = off;
        off += r.args.size();
        off = align256(off);
        r.off_bstart = off;
        off += r.bstart.size() * sizeof(int);
        off = align256(off);
        r.off_next = off;
        off += sizeof(int);
    }
    if (off > SERVER_TAB_BYTES) return MHD_ENOMEM;
    char* h = sv->htab + (size_t)half * SERVER_TAB_BYTES;
    char* d = sv->dtab + (size_t)half * SERVER_TAB_BYTES;
    for (MultiRec& r : sv->recs) {
        memcpy(h + r.off_args, r.args.data(), r.args.size());
        memcpy(h + r.off_bstart, r.bstart.data(), r.bstart.size() * sizeof(int));
        memset(h + r.off_next, 0, sizeof(int));
    }
    if (hipMemcpyAsync(d, h, off, hipMemcpyHostToDevice, sv->s) != hipSuccess) return MHD_EDEVICE;
    int nbox = (int)sv->active.size();
    for (MultiRec& r : sv->recs) {
        if (r.total == 0) continue;
        const int* bs = reinterpret_cast<const int*>(d + r.off_bstart);
        if (sv->p.persistent) {
            int st = r.go_persist(d + r.off_args, bs, nbox, r.total, r.shm, sv->s, sv->ncu, sv->p.max_workgroups,
                                  reinterpret_cast<int*>(d + r.off_next));
            if (st) return st;
        } else {
            r.go(d + r.off_args, bs, nbox, r.total, r.shm, sv->s);
        }
    }
    return launch_status();
}

// the round in the form that fits the boxes in flight
template <typename T>
int server_round(mhd_server* sv, int half)
{
    bool far = false;
    double cells = 0.0;
    for (const mhd_server::Active& a : sv->active) {
        far = far || wide_fields(a.box);
        cells += (double)a.box->g.n;
    }
    if (far) return server_step<T, Far>(sv, half);
    return streamed(cells * sizeof(T)) ? server_step<T, Streamed>(sv, half) : server_step<T, Near>(sv, half);
}

double* ret_slot(mhd_server* sv, int half, int k)
{
    return reinterpret_cast<double*>(sv->htab + 2 * SERVER_TAB_BYTES +
                                     ((size_t)half * SERVER_MAX_SLOTS + k) * SERVER_RET_BYTES);
}

// reports a finished box: its completion record and, where it was asked for,
// its state.  On a failure nothing has changed.
int server_report(mhd_server* sv, const mhd_server::Finished& f)
{
    const mhd_server::Active& a = f.a;
    mhd_completion c;
    memset(&c, 0, sizeof(c));
    c.id = a.id;
    c.steps = a.done;
    c.t_submit = a.t_submit;
    c.t_admit = a.t_admit;
    c.cells = (int64_t)a.box->g.n;
    c.bytes = a.bytes;
    memcpy(c.totals, f.totals, sizeof(f.totals));
    c.status = flags_status(f.flags);
    HostState buf;
    if (a.keep) {
        // the kept state is copied out before the box's memory is released
        if (!buf.resize((size_t)NF * a.box->g.n)) return MHD_ENOMEM;
        const int st = sv->p.precision == MHD_FP64 ? get_f64<double>(a.box, sv->ring, buf.v.get())
                                                   : get_f64<float>(a.box, sv->ring, buf.v.get());
        if (st != MHD_OK && st != c.status) return st;
    }
    c.t_done = now_s() - sv->t0;
    try {
        sv->done.push_back(c);
    } catch (const std::bad_alloc&) {
        return MHD_ENOMEM;
    }
    if (a.keep) {
        try {
            std::swap(sv->results[a.id], buf);
        } catch (const std::bad_alloc&) {
            sv->done.pop_back();
            return MHD_ENOMEM;
        }
        pool_free(sv, a.off, a.bytes);
    }
    delete a.box;
    return MHD_OK;
}

int server_progress(mhd_server* sv, int* nact, int* npend)
{
    int st = server_admit(sv);
    if (st) return st;
    const int half = (int)(sv->rounds & 1);
    bool launched = false;
    if (!sv->active.empty()) {
        std::list<mhd_server::Finished> last;   // the boxes that this round finishes
        try {
            for (const mhd_server::Active& a : sv->active)
                if (a.done + 1 >= a.steps) last.emplace_back();
        } catch (const std::bad_alloc&) {
            return MHD_ENOMEM;
        }
        st = sv->p.precision == MHD_FP64 ? server_round<double>(sv, half) : server_round<float>(sv, half);
        if (st) return st;
        // boxes that have run their steps leave the round: their totals and
        // flags go to pinned slots behind the round on the stream, and (unless
        // their state is kept) their memory returns to the pool at once, since
        // anything that reuses it is queued behind
        int k = 0;
        for (mhd_server::Active& a : sv->active) {
            if (a.done + 1 < a.steps) continue;
            double* slot = ret_slot(sv, half, k++);
            int s2 = sv->p.precision == MHD_FP64 ? totals_launch<double>(a.box) : totals_launch<float>(a.box);
            if (s2 ||
                hipMemcpyAsync(slot, a.box->tot_dev, NF * sizeof(double), hipMemcpyDeviceToHost, sv->s) != hipSuccess ||
                hipMemcpyAsync(slot + NF, a.box->flags, sizeof(uint32_t), hipMemcpyDeviceToHost, sv->s) != hipSuccess)
                return MHD_EDEVICE;
        }
        if (hipEventRecord(sv->ev[half], sv->s) != hipSuccess) return MHD_EDEVICE;
        size_t stay = 0;
        auto f = last.begin();
        for (mhd_server::Active& a : sv->active) {
            if (++a.done < a.steps) {
                sv->active[stay++] = a;
                continue;
            }
            (f++)->a = a;
            if (!a.keep) pool_free(sv, a.off, a.bytes);
        }
        sv->active.resize(stay);
        sv->retiring[half].swap(last);
        sv->rounds++;
        launched = true;
    }
    if (nact) *nact = (int)sv->active.size();
    if (npend) *npend = (int)sv->pending.size();
    // the previous round: wait for it and take its boxes' totals and flags (the
    // slots are written again by the round after the one just launched)
    if (sv->prev_launched) {
        const int ph = half ^ 1;   // round rounds - 1 (launched by the previous call)
        if (hipEventSynchronize(sv->ev[ph]) != hipSuccess) return MHD_EDEVICE;
        int k = 0;
        for (mhd_server::Finished& f : sv->retiring[ph]) {
            const double* slot = ret_slot(sv, ph, k++);
            memcpy(f.totals, slot, sizeof(f.totals));
            memcpy(&f.flags, slot + NF, sizeof(f.flags));
        }
        sv->finished.splice(sv->finished.end(), sv->retiring[ph]);
    }
    sv->prev_launched = launched;
    while (!sv->finished.empty()) {
        st = server_report(sv, sv->finished.front());
        if (st) return st;
        sv->finished.pop_front();
    }
    return MHD_OK;
}

}  // namespace

// ---------------------------------------------------------------- C ABI

// ---------------------------------------------------------------- allocation-free totals

// Partial sums of mhd_conserved_totals_noalloc: NF doubles per chunk (44 KiB).
// Each device that loads the library holds its own copy until the process
// ends.  Host code never passes the array's name to a kernel (on the host it
// is a stand-in, not a device address): it uses the address that
// hipGetSymbolAddress returned for the current device.
static __device__ __align__(256) double scratch[(size_t)TOTALS_CHUNKS * NF];

namespace {

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[NOALLOC_MAX_DEVICES];

// device address of this device's scratch array, looked up once per device
// with that device current
int scratch_of_current_device(double** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= NOALLOC_MAX_DEVICES) return MHD_EDEVICE;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return MHD_EDEVICE;
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    *out = g_scratch_ptr[dev];
    return MHD_OK;
}

template <typename T>
int totals_noalloc(const void* state, int n, hipStream_t s, double* part, double* out)
{
    CFields<T> u;
    for (int f = 0; f < NF; f++) u.f[f] = static_cast<const T*>(state) + (size_t)f * (size_t)n;
    return totals_run<T>(u, n, s, part, out);
}

}  // namespace

extern "C" {

size_t mhd_workspace_bytes(const mhd_params* p)
{
    if (!valid_params(p)) return 0;
    return layout_of(p->n, p->precision, p->grav_G > 0.0, p->ionisation != 0).total;
}

int mhd_create(const mhd_params* p, mhd_box** out)
{
    if (!out) return MHD_EINVAL;
    *out = nullptr;
    if (!valid_params(p)) return MHD_EINVAL;
    Layout L = layout_of(p->n, p->precision, p->grav_G > 0.0, p->ionisation != 0);
    if (!p->workspace || p->workspace_bytes < L.total) return MHD_ENOMEM;
    if (((uintptr_t)p->workspace) & 255) return MHD_EINVAL;
    mhd_box* b = new (std::nothrow) mhd_box;
    if (!b) return MHD_ENOMEM;
    box_bind(b, p, L);
    *out = b;
    return MHD_OK;
}

int mhd_set_timing(mhd_box* b, int enable)
{
    if (!b) return MHD_EINVAL;
    if (enable && !b->ev_ready) {
        for (int i = 0; i < 2 * EVCAP; i++)
            if (hipEventCreate(&b->ev[i]) != hipSuccess) return MHD_EDEVICE;
        b->ev_ready = 1;
    }
    b->timing = enable ? 1 : 0;
    b->nev = 0;
    for (int c = 0; c < MHD_NKCLASS; c++) {
        b->tms[c] = 0.0;
        b->tcnt[c] = 0;
    }
    return MHD_OK;
}

int mhd_get_timing(mhd_box* b, double* ms, int64_t* counts)
{
    if (!b || !ms || !counts) return MHD_EINVAL;
    int st = timing_collect(b);
    if (st) return st;
    for (int c = 0; c < MHD_NKCLASS; c++) {
        ms[c] = b->tms[c];
        counts[c] = b->tcnt[c];
    }
    return MHD_OK;
}

int mhd_init_state(mhd_box* b, const double* prim)
{
    if (!b || !prim) return MHD_EINVAL;
    return b->prec == MHD_FP64 ? load_f64<double>(b, prim, true) : load_f64<float>(b, prim, true);
}

int mhd_set_state(mhd_box* b, const double* cons)
{
    if (!b || !cons) return MHD_EINVAL;
    return b->prec == MHD_FP64 ? load_f64<double>(b, cons, false) : load_f64<float>(b, cons, false);
}

int mhd_get_state(mhd_box* b, double* cons_out)
{
    if (!b || !cons_out) return MHD_EINVAL;
    return b->prec == MHD_FP64 ? get_f64<double>(b, b->ring, cons_out) : get_f64<float>(b, b->ring, cons_out);
}

int mhd_get_potential(mhd_box* b, double* phi_out)
{
    if (!b || !phi_out || !b->grav) return MHD_EINVAL;
    OneEmit<Near> e{ b };   // the Poisson kernels index by cell
    const size_t N = (size_t)b->g.n;
    if (b->prec == MHD_FP64) {
        emit_poisson<double>(b, e);
        if (launch_status()) return MHD_EDEVICE;
        if (hipMemcpyAsync(phi_out, b->phi, N * 8, hipMemcpyDeviceToHost, b->s) != hipSuccess) return MHD_EDEVICE;
        return sync_and_flags(b);
    }
    emit_poisson<float>(b, e);
    if (launch_status()) return MHD_EDEVICE;
    std::vector<float> tmp(N);
    if (hipMemcpyAsync(tmp.data(), b->phi, N * 4, hipMemcpyDeviceToHost, b->s) != hipSuccess) return MHD_EDEVICE;
    int st = sync_and_flags(b);
    for (size_t c = 0; c < N; c++) phi_out[c] = (double)tmp[c];
    return st;
}

int mhd_cfl_dt(mhd_box* b, double* dt_out)
{
    if (!b || !dt_out) return MHD_EINVAL;
    if (hipMemcpyAsync(dt_out, b->dt_dev, sizeof(double), hipMemcpyDeviceToHost, b->s) != hipSuccess)
        return MHD_EDEVICE;
    return sync_and_flags(b);
}

int mhd_step(mhd_box* b, double dt)
{
    if (!b || !std::isfinite(dt) || !(dt > 0.0)) return MHD_EINVAL;
    return b->prec == MHD_FP64 ? full_step<double>(b, dt, false) : full_step<float>(b, dt, false);
}

int mhd_step_cfl(mhd_box* b)
{
    if (!b) return MHD_EINVAL;
    return b->prec == MHD_FP64 ? full_step<double>(b, 0.0, true) : full_step<float>(b, 0.0, true);
}

int mhd_conserved_totals(mhd_box* b, double out[MHD_NFIELDS])
{
    if (!b || !out) return MHD_EINVAL;
    return b->prec == MHD_FP64 ? totals<double>(b, out) : totals<float>(b, out);
}

int mhd_conserved_totals_noalloc(const void* state, int32_t precision, const int32_t n[3], void* stream,
                                 double* out)
{
    if (!state || !n || !out || (precision != MHD_FP64 && precision != MHD_FP32_MIXED)) return MHD_EINVAL;
    if (!valid_dims(n)) return MHD_EINVAL;
    const int64_t cells = (int64_t)n[0] * n[1] * n[2];
    if (cells > MHD_NOALLOC_MAX_CELLS) return MHD_ETOOLARGE;
    double* part = nullptr;
    int st = scratch_of_current_device(&part);
    if (st) return st;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    return precision == MHD_FP64 ? totals_noalloc<double>(state, (int)cells, s, part, out)
                                 : totals_noalloc<float>(state, (int)cells, s, part, out);
}

int mhd_debug_stage(mhd_box* b, int stage, double dt)
{
    if (!b) return MHD_EINVAL;
    if (stage != MHD_STAGE_TAIL && (!std::isfinite(dt) || !(dt > 0.0))) return MHD_EINVAL;
    if (stage == MHD_STAGE_TAIL && (!std::isfinite(dt) || dt < 0.0)) return MHD_EINVAL;
    return b->prec == MHD_FP64 ? debug_stage<double>(b, stage, dt) : debug_stage<float>(b, stage, dt);
}

int mhd_destroy(mhd_box* b)
{
    if (b && b->ev_ready)
        for (int i = 0; i < 2 * EVCAP; i++) (void)hipEventDestroy(b->ev[i]);
    if (b) ring_release(b->ring);
    delete b;
    return MHD_OK;
}

const char* mhd_strerror(int status)
{
    switch (status) {
    case MHD_OK: return "ok";
    case MHD_EINVAL: return "invalid argument";
    case MHD_ENOMEM: return "workspace missing or too small, or no host memory";
    case MHD_EDEVICE: return "HIP runtime error";
    case MHD_ECFL: return "time step above the CFL bound";
    case MHD_ENONPHYS: return "non-finite or non-positive density or internal energy";
    case MHD_ETOOLARGE: return "box larger than the allocation-free entry point (on static scratch) takes";
    default: return "unknown status";
    }
}

size_t mhd_server_reserved_bytes(void) { return 2 * SERVER_TAB_BYTES; }

size_t mhd_server_box_bytes(const mhd_server_params* p, const int32_t n[3])
{
    if (!p || !n || !valid_dims(n)) return 0;
    if (p->precision != MHD_FP64 && p->precision != MHD_FP32_MIXED) return 0;
    return align256(layout_of(n, p->precision, false, false).total);
}

int mhd_server_create(const mhd_server_params* p, mhd_server** out)
{
    if (!out) return MHD_EINVAL;
    *out = nullptr;
    if (!p) return MHD_EINVAL;
    if (!valid_physics(p->precision, p->gamma, p->cfl, p->theta, p->chemistry, p->cooling, p->n_unit_cm3,
                       p->T_unit_K, p->t_unit_s))
        return MHD_EINVAL;
    if (p->max_slots < 1 || p->max_slots > SERVER_MAX_SLOTS) return MHD_EINVAL;
    if (p->persistent != 0 && p->persistent != 1) return MHD_EINVAL;
    if (p->max_workgroups < 0) return MHD_EINVAL;
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
        return MHD_EDEVICE;
    if (!p->workspace || p->workspace_bytes < 2 * SERVER_TAB_BYTES + 4096) return MHD_ENOMEM;
    if (((uintptr_t)p->workspace) & 255) return MHD_EINVAL;
    mhd_server* sv = new (std::nothrow) mhd_server;
    if (!sv) return MHD_ENOMEM;
    sv->p = *p;
    sv->s = reinterpret_cast<hipStream_t>(p->stream);
    sv->dtab = reinterpret_cast<char*>(p->workspace);
    sv->pool = sv->dtab + 2 * SERVER_TAB_BYTES;
    sv->pool_bytes = (p->workspace_bytes - 2 * SERVER_TAB_BYTES) & ~(size_t)255;
    sv->freel.push_back(std::make_pair((size_t)0, sv->pool_bytes));
    sv->used = sv->peak = 0;
    sv->next_id = 1;
    sv->t0 = now_s();
    sv->htab = nullptr;
    sv->rounds = 0;
    sv->ncu = ncu;
    sv->prev_launched = false;
    sv->ev_ready = 0;
    if (hipHostMalloc(reinterpret_cast<void**>(&sv->htab), SERVER_HOST_BYTES, hipHostMallocDefault) != hipSuccess) {
        delete sv;
        return MHD_EDEVICE;
    }
    if (hipEventCreateWithFlags(&sv->ev[0], hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&sv->ev[1], hipEventDisableTiming) != hipSuccess) {
        (void)hipHostFree(sv->htab);
        delete sv;
        return MHD_EDEVICE;
    }
    sv->ev_ready = 1;
    *out = sv;
    return MHD_OK;
}

int mhd_server_submit(mhd_server* sv, const mhd_request* r, const double* prim, uint64_t* id)
{
    if (!sv || !r || !prim || !id) return MHD_EINVAL;
    if (!valid_dims(r->n) || r->steps < 1) return MHD_EINVAL;
    if (r->n[0] > SERVER_MAX_NX) return MHD_EINVAL;
    if (align256(layout_of(r->n, sv->p.precision, false, false).total) > sv->pool_bytes) return MHD_ENOMEM;
    mhd_server::Pending q;
    if (r->borrow != 0 && r->borrow != 1) return MHD_EINVAL;
    q.id = sv->next_id++;
    q.r = *r;
    size_t n = (size_t)r->n[0] * r->n[1] * r->n[2];
    if (r->borrow)
        q.src = prim;
    else
    {
        if (!q.prim.resize((size_t)MHD_NPRIM * n)) return MHD_ENOMEM;
        host_copy(q.prim.v.get(), prim, q.prim.n * sizeof(double));
    }
    q.t_submit = now_s() - sv->t0;
    sv->pending.push_back(std::move(q));
    *id = sv->pending.back().id;
    return MHD_OK;
}

int mhd_server_progress(mhd_server* sv, int* n_active, int* n_pending)
{
    if (!sv) return MHD_EINVAL;
    return server_progress(sv, n_active, n_pending);
}

int mhd_server_poll(mhd_server* sv, mhd_completion* out, int cap, int* n)
{
    if (!sv || !n || (cap > 0 && !out)) return MHD_EINVAL;
    int k = 0;
    while (k < cap && !sv->done.empty()) {
        out[k++] = sv->done.front();
        sv->done.pop_front();
    }
    *n = k;
    return MHD_OK;
}

int mhd_server_result(mhd_server* sv, uint64_t id, double* cons_out, size_t count)
{
    if (!sv || !cons_out) return MHD_EINVAL;
    auto it = sv->results.find(id);
    if (it == sv->results.end()) return MHD_EINVAL;
    if (count != it->second.n) return MHD_EINVAL;
    host_copy(cons_out, it->second.v.get(), count * sizeof(double));
    sv->results.erase(it);
    return MHD_OK;
}

int mhd_server_memory(mhd_server* sv, size_t* used, size_t* peak, size_t* capacity)
{
    if (!sv) return MHD_EINVAL;
    if (used) *used = sv->used;
    if (peak) *peak = sv->peak;
    if (capacity) *capacity = sv->pool_bytes;
    return MHD_OK;
}

int mhd_server_destroy(mhd_server* sv)
{
    if (!sv) return MHD_OK;
    (void)hipStreamSynchronize(sv->s);
    for (mhd_server::Active& a : sv->active) delete a.box;
    for (const std::list<mhd_server::Finished>* l : { &sv->retiring[0], &sv->retiring[1], &sv->finished })
        for (const mhd_server::Finished& f : *l) delete f.a.box;
    if (sv->ev_ready) {
        (void)hipEventDestroy(sv->ev[0]);
        (void)hipEventDestroy(sv->ev[1]);
    }
    if (sv->htab) (void)hipHostFree(sv->htab);
    ring_release(sv->ring);
    delete sv;
    return MHD_OK;
}

}  // extern "C"
