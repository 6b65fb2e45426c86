// Forward sampling (paper Eq. 2 with the cutoff test of Sec. 4.1.1 and the
// definedness rule of Sec. 4.1.3).
//
// The whitened offset u = U (p - mu) of a (Gaussian, query) pair is linear in
// the query: with offsets a = p - o from a point o of the cell and c = U (mu
// - o), u = U a - c is a product of the 3 x 4 matrix (-c, U) with (1, a). For
// 16 queries and 16 Gaussians these are three 16x16x4 float32 matrix
// products (v_mfma_f32_16x16x4_f32), each component an ascending chain of
// float32 fused multiply-adds. They do not run beside vector work (measured: 36
// cycles each, added to the vector instructions' time), so they cost 27 issue
// slots per 256 pairs where the vector form takes 24; what they save is the
// vector form's read of every record from LDS once per 64 queries, which bounds
// it (24 LDS cycles a record and wave, four SIMDs to an LDS).
// The walk of dense cells in boxed launches takes them (k_sample_dense).
//
// Grid queries (Sec. 4.1.3, Fig. 4 C): one wavefront per (cell, 64 voxels of
// the cell), a voxel a lane; cells of at most 64 voxels split the list over
// the lanes (walk_split).
//
// Voxel-list, point and jittered queries (Sec. 5.1.2): the queries are first
// ordered by cell and, inside a cell, by quarter of the cell along x
// (query_keys + radix sort, kept in the plan), and the work is split by cell
// (see k_sample_cells). Where many queries meet long lists (boxed_list), the
// forward also orders them by place inside the quarter (k_refine_order) and
// cuts dense cells into boxes that meet only the candidates reaching them
// (k_sample_dense).
#include "expand.h"
#include "internal.h"
#include "radix.h"

#pragma clang fp contract(off)

namespace gs {

namespace {


// The samplers run one wave per workgroup. Their waves are independent
// (each has its own LDS buffer) and the cost of a work item varies by
// orders of magnitude with the cell's list and queries: a workgroup keeps
// its LDS until its slowest wave ends, so one-wave workgroups hand a
// finished wave's slot and LDS straight to new work. Work items are taken
// in launch order, which the dispatcher deals round-robin over the XCDs:
// with a fixed block-to-XCD remap, each XCD would own one contiguous
// stretch of cells, and clustered data would leave most XCDs idle while
// one works through the dense part.
constexpr int kSampWaves = 1;
constexpr int kSampBlock = kSampWaves * kWave;
// Waves per SIMD the samplers are compiled for.
constexpr int kSampPerSimd = 7;

// Q' = Q log2(e) / 2 of a record at a point (record_q), G = 2^-Q'.
__device__ __forceinline__ float cutoff_q(const Record &r, float px, float py, float pz) {
    return record_q(r, px, py, pz);
}

__device__ __forceinline__ void accumulate(const Record &r, float px, float py, float pz, float T, float &I,
                                           float &V) {
    const float Q = cutoff_q(r, px, py, pz);
    if (Q <= T) {
        const float G = exp2_hw(-Q);
        I = fmaf_(r.f0.w, G, I);
        V = fmaf_(r.f1.w, G, V);
    }
}

// c = U (mu - o) of a record, formed in float64 and rounded once.
__device__ __forceinline__ void centre_offset(const Record &r, float ox, float oy, float oz, float (&c)[3]) {
    const double bx = (double)r.f0.x - (double)ox, by = (double)r.f0.y - (double)oy, bz = (double)r.f0.z - (double)oz;
    c[0] = (float)((double)r.f1.x * bx + ((double)r.f1.y * by + (double)r.f1.z * bz));
    c[1] = (float)((double)r.f2.x * by + (double)r.f2.y * bz);
    c[2] = (float)((double)r.f2.z * bz);
}

// Records staged for the queries of one cell are rewritten relative to a
// point o of the cell (its centre): the first quarter of candidate s holds
// (-c, w) with c = U (mu - o), so that a query at a = p - o has u = U a - c,
// six FMAs where U (p - mu) takes three subtractions and six operations.
// Both offsets are at most a cell and a cutoff radius long, so u is formed
// from terms of its own size plus the cell's extent in units of the
// Gaussian's scale, and the rounding of Q' grows with that extent: on the
// five workloads' Gaussians near their cutoffs it stays within 0.15 of the
// float32 band of the cutoff the oracle allows (0.07 for U (p - mu)), but
// with cells a few hundred times a Gaussian's largest scale it leaves the
// band. The preprocess marks the cells of such Gaussians' boxes (cell
// diagonal above kOffsetCells times the largest scale), and the dense walk
// evaluates a marked cell as U (p - mu).
// Lane s rewrites candidate s of the wave's planes. The dense cells' walk
// takes it: with two queries a lane it is bound by VALU issue (10^8
// clustered points, before they were boxed: the forward 6.6 % faster), and the
// items of one query a lane take it too so that both give the same bits, which
// are also the boxed walk's (stage_rows). The query rows are bound by their
// LDS reads, and the rewrite made them 1-3 % slower; they keep U (p - mu). So
// do the grid cells: the backward's sets are formed by it, and what rounds does
// not grow with the cell (walk_split).
__device__ __forceinline__ void offset_planes(float4 *buf, uint32_t lane, float ox, float oy, float oz) {
    Record r;
    r.f0 = buf[lane];
    r.f1 = buf[kWave + lane];
    r.f2 = buf[2 * kWave + lane];
    float c[3];
    centre_offset(r, ox, oy, oz, c);
    buf[lane] = make_float4(-c[0], -c[1], -c[2], r.f0.w);
}

// Q' of a rewritten record (f0 = (-c, w)) at the offset a = p - o.
__device__ __forceinline__ float offset_q(const Record &r, float ax, float ay, float az) {
    const float u0 = fmaf_(r.f1.x, ax, fmaf_(r.f1.y, ay, fmaf_(r.f1.z, az, r.f0.x)));
    const float u1 = fmaf_(r.f2.x, ay, fmaf_(r.f2.y, az, r.f0.y));
    const float u2 = fmaf_(r.f2.z, az, r.f0.z);
    return fmaf_(u0, u0, fmaf_(u1, u1, u2 * u2));
}

// The sums without a branch: G is selected (0 past the cutoff) and always
// added, so that a lane's queries cost one select each (adding w 0 and
// (w v) 0 leaves I and V as they are: both start at +0 and w, v are finite).
__device__ __forceinline__ void accumulate_sel(const Record &r, float px, float py, float pz, float T, float &I,
                                               float &V) {
    const float Q = cutoff_q(r, px, py, pz);
    const float G = Q <= T ? exp2_hw(-Q) : 0.0f;
    I = fmaf_(r.f0.w, G, I);
    V = fmaf_(r.f1.w, G, V);
}

__device__ __forceinline__ void accumulate_off_sel(const Record &r, float ax, float ay, float az, float T, float &I,
                                                   float &V) {
    const float Q = offset_q(r, ax, ay, az);
    const float G = Q <= T ? exp2_hw(-Q) : 0.0f;
    I = fmaf_(r.f0.w, G, I);
    V = fmaf_(r.f1.w, G, V);
}

// Four consecutive work items per XCD (xcd_group): the items of one cell
// share that XCD's L2 (C5's forward 1.6 % faster, C4's unchanged).
constexpr uint32_t kXcdItems = 4;

// The centre of cell c (float32; any point of the cell would do), for a
// wave-uniform c: kept in scalar registers.
__device__ __forceinline__ void cell_centre(const GridParams &g, uint32_t c, float &ox, float &oy, float &oz) {
    const uint32_t nx = (uint32_t)g.cells[0], ny = (uint32_t)g.cells[1];
    const uint32_t cx = c % nx, cy = (c / nx) % ny, cz = c / (nx * ny);
    ox = readfirst_f(g.lo[0] + ((float)cx + 0.5f) / g.invc[0]);
    oy = readfirst_f(g.lo[1] + ((float)cy + 0.5f) / g.invc[1]);
    oz = readfirst_f(g.lo[2] + ((float)cz + 0.5f) / g.invc[2]);
}

constexpr int kDenseWaves = kWavesPerBlock;  // waves of a dense item's workgroup
// Waves per SIMD (its LDS holds six workgroups a CU). A bound also keeps the
// matrix products' results in ordinary registers: with the whole register file
// to itself the compiler puts them in accumulation registers and moves each
// out again.
constexpr int kDensePerSimd = 6;
constexpr uint32_t kTile = 16;              // queries of a matrix tile, and Gaussians

// LDS of a dense item's workgroup. The records of up to kBlock candidates:
// the rows (-c_i, U_iz, U_iy, U_ix) of (-c, U), in the order the matrix
// product's fused multiply-adds take them, and (w, w v). -c comes first, so
// that Q' has offset_q's bits. (c last, the sums of U a are rounded by
// themselves before c cancels them: 1.0 to 1.4 times the rms error of Q' at the
// cutoff, round Gaussians in cells of 6 to 60 times their scale.) Entry kBlock
// is an all-zero record that pads lists to whole tiles. The walk of a coarse
// cell uses the rows' space for staged records, a quarter of it a wave
// (wave_records).
struct DenseLds {
    float4 b[3][kBlock + 1];
    float2 w[kBlock];
    // each wave's list of the candidates that reach its queries: their
    // entries, and their weights in list order
    uint16_t list[kDenseWaves][kBlock + kTile];
    float lw[kDenseWaves][kBlock + kTile], lv[kDenseWaves][kBlock + kTile];
    uint16_t tile_start[kBlock], tile_bin[kBlock];
    uint64_t ballot[2][kDenseWaves];
    uint32_t next;
};
static_assert(sizeof(float4) * kRecordQuads * kWave * kDenseWaves <= sizeof(DenseLds::b), "staged records fit the rows");

__device__ __forceinline__ float4 *wave_records(DenseLds &L, uint32_t wave) {
    return &L.b[0][0] + kRecordQuads * kWave * wave;
}

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ Record load_record(const Record *__restrict__ rec, uint32_t g) {
    const float4 *p = (const float4 *)(rec + g);
    Record r;
    r.f0 = p[0];
    r.f1 = p[1];
    r.f2 = p[2];
    return r;
}

// A candidate's rows into entry b[0] of planes `plane` entries apart: record
// r about o, or the all-zero record.
__device__ __forceinline__ void stage_rows(float4 *b, uint32_t plane, bool live, const Record &r, float ox, float oy,
                                           float oz) {
    float4 b0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b1 = b0, b2 = b0;
    if (live) {
        float c[3];
        centre_offset(r, ox, oy, oz, c);
        b0 = make_float4(-c[0], r.f1.z, r.f1.y, r.f1.x);
        b1 = make_float4(-c[1], r.f2.y, r.f2.x, 0.0f);
        b2 = make_float4(-c[2], r.f2.z, 0.0f, 0.0f);
    }
    b[0] = b0;
    b[plane] = b1;
    b[2 * plane] = b2;
}

// Operand of the matrix products that holds a tile's queries: lane l has
// component l / 16 of (1, a_z, a_y, a_x) for query l % 16.
__device__ __forceinline__ float tile_operand(uint32_t k, float ax, float ay, float az) {
    return k == 0 ? 1.0f : (k == 1 ? az : (k == 2 ? ay : ax));
}

// The 256 pairs of 16 candidates (operands g0, g1, g2: lane l has component
// l / 16 of the rows of candidate l % 16) and one tile of queries (operand q).
// Lane l gets the pairs of query l % 16 with candidates 4 (l / 16) + r, r < 4,
// whose weights are w[r] and v[r], and adds them to its sums.
__device__ __forceinline__ void tile_pairs(float q, float g0, float g1, float g2, const float4 &w, const float4 &v,
                                           float T, float &I, float &V) {
    const mfma_f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const mfma_f4 u0 = __builtin_amdgcn_mfma_f32_16x16x4f32(g0, q, zero, 0, 0, 0);
    const mfma_f4 u1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g1, q, zero, 0, 0, 0);
    const mfma_f4 u2 = __builtin_amdgcn_mfma_f32_16x16x4f32(g2, q, zero, 0, 0, 0);
    const float wr[4] = {w.x, w.y, w.z, w.w}, vr[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float Q = fmaf_(u0[r], u0[r], fmaf_(u1[r], u1[r], u2[r] * u2[r]));
        // selected, not branched: adding w 0 and (w v) 0 leaves the sums as
        // they are (they start at +0; w and v are finite)
        const float G = Q <= T ? exp2_hw(-Q) : 0.0f;
        I = fmaf_(wr[r], G, I);
        V = fmaf_(vr[r], G, V);
    }
}

// a and b, each a sum per lane, added over the wave's halves: lanes 0..31 get
// a's totals of lanes l and l + 32, lanes 32..63 b's.
__device__ __forceinline__ float swap32_sum(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The same over the rows of 16 of each half: even rows get a's, odd rows b's.
__device__ __forceinline__ float swap16_sum(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Tile t's sums over its candidates for t < 4: lane l gets those of query
// l % 16 of tile l / 16.
__device__ __forceinline__ float tile_sum(float t0, float t1, float t2, float t3) {
    return swap16_sum(swap32_sum(t0, t2), swap32_sum(t1, t3));
}

// Walk a wave-uniform candidate list [ja, jb) for one query per lane. The
// list is staged in the wave's LDS planes (buf: 3 planes of kWave float4) 64
// records at a time: lane l copies candidate c0 + l's record from memory
// straight into LDS (lanes past the list copy its last record), the ids of
// the next 64 are fetched meanwhile, and every lane then reads each record
// with the same address (a broadcast). One wait for memory per 64
// candidates, instead of a dependent id and record load per candidate.
__device__ __forceinline__ void walk_staged(const Record *__restrict__ rec, const uint32_t *__restrict__ gids,
                                            uint32_t ja, uint32_t jb, uint32_t lane, float4 *buf, float px,
                                            float py, float pz, float T, float &I, float &V) {
    uint32_t gnext = 0;
    if (ja < jb) gnext = gids[ja + lane < jb ? ja + lane : jb - 1];
    for (uint32_t c0 = ja; c0 < jb; c0 += kWave) {
        const float4 *src = (const float4 *)(rec + gnext);
#pragma unroll
        for (int qq = 0; qq < kRecordQuads; ++qq)
            __builtin_amdgcn_global_load_lds((const void *)(src + qq),
                                             (__attribute__((address_space(3))) void *)(buf + qq * kWave), 16, 0, 0);
        if (c0 + kWave < jb) gnext = gids[c0 + kWave + lane < jb ? c0 + kWave + lane : jb - 1];
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
        const uint32_t cnt = jb - c0 < (uint32_t)kWave ? jb - c0 : (uint32_t)kWave;
        uint32_t s = 0;
        for (; s + 2 <= cnt; s += 2) {
            Record a, b;
            a.f0 = buf[s];
            a.f1 = buf[kWave + s];
            a.f2 = buf[2 * kWave + s];
            b.f0 = buf[s + 1];
            b.f1 = buf[kWave + s + 1];
            b.f2 = buf[2 * kWave + s + 1];
            accumulate(a, px, py, pz, T, I, V);
            accumulate(b, px, py, pz, T, I, V);
        }
        if (s < cnt) {
            Record a;
            a.f0 = buf[s];
            a.f1 = buf[kWave + s];
            a.f2 = buf[2 * kWave + s];
            accumulate(a, px, py, pz, T, I, V);
        }
        // every lane has read the planes before the next chunk overwrites them
        __builtin_amdgcn_wave_barrier();
    }
}

// R queries per lane against a wave-uniform list [ja, jb), staged in the
// wave's LDS planes 64 records at a time as in walk_staged: each record
// read there serves the lane's R queries.
template <uint32_t R>
__device__ __forceinline__ void walk_staged_r(const Record *__restrict__ rec, bool off,
                                              const uint32_t *__restrict__ gids, uint32_t ja, uint32_t jb,
                                              uint32_t lane, float4 *buf,
                                              const float (&px)[R], const float (&py)[R], const float (&pz)[R],
                                              float ox, float oy, float oz, float T, float (&I)[R],
                                              float (&V)[R]) {
    float ax[R], ay[R], az[R];
#pragma unroll
    for (uint32_t t = 0; t < R; ++t) {
        ax[t] = px[t] - ox;
        ay[t] = py[t] - oy;
        az[t] = pz[t] - oz;
    }
    uint32_t gnext = 0;
    if (ja < jb) gnext = gids[ja + lane < jb ? ja + lane : jb - 1];
    for (uint32_t c0 = ja; c0 < jb; c0 += kWave) {
        const float4 *src = (const float4 *)(rec + gnext);
#pragma unroll
        for (int qq = 0; qq < kRecordQuads; ++qq)
            __builtin_amdgcn_global_load_lds((const void *)(src + qq),
                                             (__attribute__((address_space(3))) void *)(buf + qq * kWave), 16, 0, 0);
        if (c0 + kWave < jb) gnext = gids[c0 + kWave + lane < jb ? c0 + kWave + lane : jb - 1];
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
        const uint32_t cnt = jb - c0 < (uint32_t)kWave ? jb - c0 : (uint32_t)kWave;
        if (off) {
            // every record of the chunk rewritten to offsets from o
            offset_planes(buf, lane, ox, oy, oz);
            __builtin_amdgcn_wave_barrier();
            for (uint32_t s = 0; s < cnt; ++s) {
                Record a;
                a.f0 = buf[s];
                a.f1 = buf[kWave + s];
                a.f2 = buf[2 * kWave + s];
#pragma unroll
                for (uint32_t t = 0; t < R; ++t) accumulate_off_sel(a, ax[t], ay[t], az[t], T, I[t], V[t]);
            }
        } else {
            // a cell that may list a coarse Gaussian: U (p - mu)
            for (uint32_t s = 0; s < cnt; ++s) {
                Record a;
                a.f0 = buf[s];
                a.f1 = buf[kWave + s];
                a.f2 = buf[2 * kWave + s];
#pragma unroll
                for (uint32_t t = 0; t < R; ++t) accumulate_sel(a, px[t], py[t], pz[t], T, I[t], V[t]);
            }
        }
        // every lane has read the planes before the next chunk overwrites them
        __builtin_amdgcn_wave_barrier();
    }
}


// walk_staged for a cell of at most 64 voxels, lane l at (px, py, pz) of voxel
// l: SL lanes a voxel and R voxels a lane, lane l testing voxels l / SL + (64 /
// SL) t, t < R, with the candidates c0 + l mod SL + SL i of each 64. With a
// voxel a lane the lanes past the cell's voxels idle through the whole list,
// and every candidate's record is read from LDS for one voxel a lane, which
// bounds the walk. 529,113 Gaussians in 58^3 cells, us, a voxel a lane and
// split: 1 voxel a cell 581 and 185, 8 voxels 523 and 202, 16 526 and 192, 32
// 528 and 260, 48 537 and 359, 64 533 and 450. (Matrix tiles take offsets from
// a point of the cell, whose rounding grows with the cell against the
// Gaussians' smallest scales, and took 248, 221, 216, 305 and 392 us up to 48
// voxels.)
template <uint32_t SL, uint32_t R>
__device__ __forceinline__ void walk_split(const Record *__restrict__ rec, const uint32_t *__restrict__ gids,
                                           uint32_t ja, uint32_t jb, uint32_t lane, float4 *buf, float px0, float py0,
                                           float pz0, float T, float &Io, float &Vo) {
    static_assert(R <= SL, "a lane of each voxel for each of a lane's voxels");
    constexpr uint32_t N = kWave / SL;  // voxels of one t
    const uint32_t slot = lane % SL;
    float px[R], py[R], pz[R], I[R], V[R];
#pragma unroll
    for (uint32_t t = 0; t < R; ++t) {
        const int src = (int)(lane / SL + N * t);
        px[t] = __shfl(px0, src, kWave);
        py[t] = __shfl(py0, src, kWave);
        pz[t] = __shfl(pz0, src, kWave);
        I[t] = V[t] = 0.0f;
    }
    uint32_t gnext = 0;
    if (ja < jb) gnext = gids[ja + lane < jb ? ja + lane : jb - 1];
    for (uint32_t c0 = ja; c0 < jb; c0 += kWave) {
        const float4 *src = (const float4 *)(rec + gnext);
#pragma unroll
        for (int qq = 0; qq < kRecordQuads; ++qq)
            __builtin_amdgcn_global_load_lds((const void *)(src + qq),
                                             (__attribute__((address_space(3))) void *)(buf + qq * kWave), 16, 0, 0);
        if (c0 + kWave < jb) gnext = gids[c0 + kWave + lane < jb ? c0 + kWave + lane : jb - 1];
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
        const uint32_t cnt = jb - c0 < (uint32_t)kWave ? jb - c0 : (uint32_t)kWave;
        for (uint32_t s0 = 0; s0 < cnt; s0 += SL) {
            const uint32_t s = s0 + slot;  // < kWave
            if (s < cnt) {
                Record a;
                a.f0 = buf[s];
                a.f1 = buf[kWave + s];
                a.f2 = buf[2 * kWave + s];
#pragma unroll
                for (uint32_t t = 0; t < R; ++t) accumulate(a, px[t], py[t], pz[t], T, I[t], V[t]);
            }
        }
        // every lane has read the planes before the next chunk overwrites them
        __builtin_amdgcn_wave_barrier();
    }
    // lane l's sums of voxel l / SL + N (l mod SL), then voxel l's to lane l
    float Is = 0.0f, Vs = 0.0f;
#pragma unroll
    for (uint32_t t = 0; t < R; ++t) {
#pragma unroll
        for (uint32_t o = 1; o < SL; o <<= 1) {
            I[t] += __shfl_xor(I[t], (int)o, kWave);
            V[t] += __shfl_xor(V[t], (int)o, kWave);
        }
        Is = slot == t ? I[t] : Is;
        Vs = slot == t ? V[t] : Vs;
    }
    const int from = (int)((lane % N) * SL + lane / N) & (kWave - 1);
    Io = __shfl(Is, from, kWave);
    Vo = __shfl(Vs, from, kWave);
}

// A wave's voxels of a grid cell, voxel first + l in lane l: all of the cell's,
// walk_split's way, or 64 of them a lane each (SL 1, walk_staged).
template <uint32_t SL, uint32_t R>
__global__ __launch_bounds__(kWave, kSampPerSimd) void k_sample_grid(QueryParams q, GridParams g,
                                                        const Record *__restrict__ rec,
                                                        const uint32_t *__restrict__ gids,
                                                        const uint32_t *__restrict__ cell_off, float T, float tau,
                                                        float *__restrict__ out_v, float *__restrict__ out_i) {
    __shared__ float4 s_rec[kRecordQuads * kWave];
    const uint32_t rx = (uint32_t)(q.dims[0] / g.cells[0]);
    const uint32_t ry = (uint32_t)(q.dims[1] / g.cells[1]);
    const uint32_t rz = (uint32_t)(q.dims[2] / g.cells[2]);
    const uint32_t vpc = rx * ry * rz;
    const uint32_t wpc = SL > 1 ? 1u : (vpc + kWave - 1) / kWave;
    const uint32_t lane = threadIdx.x;
    // ncells wpc < 2^32: at most a wave per cell and one per 64 voxels
    const uint32_t cell = blockIdx.x / wpc;
    const uint32_t local = (blockIdx.x - cell * wpc) * kWave + lane;
    const uint32_t nx = (uint32_t)g.cells[0], ny = (uint32_t)g.cells[1];
    const uint32_t cyz = cell / nx, cx = cell - cyz * nx, cz = cyz / ny, cy = cyz - cz * ny;
    const uint32_t lyz = local / rx, lx = local - lyz * rx, lz = lyz / ry, ly = lyz - lz * ry;
    const int32_t vx = (int32_t)(cx * rx + lx), vy = (int32_t)(cy * ry + ly), vz = (int32_t)(cz * rz + lz);
    const float px = voxel_center(vx, g.lo[0], q.vsz[0]);
    const float py = voxel_center(vy, g.lo[1], q.vsz[1]);
    const float pz = voxel_center(vz, g.lo[2], q.vsz[2]);
    const uint32_t j0 = ((ConstU32 *)cell_off)[cell], j1 = ((ConstU32 *)cell_off)[cell + 1];
    float I = 0.0f, V = 0.0f;
    if constexpr (SL == 1)
        walk_staged(rec, gids, j0, j1, lane, s_rec, px, py, pz, T, I, V);
    else if (j0 < j1)
        walk_split<SL, R>(rec, gids, j0, j1, lane, s_rec, px, py, pz, T, I, V);
    if (local < vpc) {
        const uint64_t idx = (uint64_t)vx + (uint64_t)q.dims[0] * ((uint64_t)vy + (uint64_t)q.dims[1] * (uint64_t)vz);
        const bool def = I > tau;
        out_v[idx] = def ? V / I : 0.0f;
        out_i[idx] = def ? I : 0.0f;
    }
}

// Sort key of query i: kSub cell + quarter of the cell along x, kSub ncells
// outside the domain.
__device__ __forceinline__ uint32_t query_key(const QueryParams &q, const GridParams &g, uint32_t i) {
    float p[3];
    bool valid;
    query_position(q, g, i, p[0], p[1], p[2], valid);
    const uint32_t outside = kSub * (uint32_t)g.ncells;
    if (!valid) return outside;
    bool inside = true;
    int64_t c[3];
    float tx = 0.0f;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        inside = inside && (p[j] >= g.lo[j]) && (p[j] <= g.hi[j]);
        const float t = (p[j] - g.lo[j]) * g.invc[j];
        int64_t ci = (int64_t)floorf(t);
        ci = ci < 0 ? 0 : ci;
        ci = ci > g.cells[j] - 1 ? g.cells[j] - 1 : ci;
        c[j] = ci;
        if (j == 0) tx = t;
    }
    if (!inside) return outside;
    // the quarter of the cell along x: floor(4 (t - c)), exact in float32 (t -
    // c is exact, the product by 4 too)
    const float fq = floorf((tx - (float)c[0]) * (float)kSub);
    const uint32_t qx = fq < 0.0f ? 0u : (fq > (float)(kSub - 1) ? kSub - 1 : (uint32_t)fq);
    return kSub * (uint32_t)(c[0] + (int64_t)g.cells[0] * (c[1] + (int64_t)g.cells[1] * c[2])) + qx;
}

__global__ __launch_bounds__(kBlock) void k_query_keys(QueryParams q, GridParams g, uint32_t *__restrict__ keys,
                                                       uint32_t *__restrict__ ids, RadixPass0 pass0) {
    __shared__ uint32_t hist_lds[kMaxDigits];
    Pass0Hist hist(hist_lds, pass0);
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int64_t i = (int64_t)blockIdx.x * kSortTile + (int64_t)it * kBlock + threadIdx.x;
        if (i < q.n) {
            const uint32_t key = query_key(q, g, (uint32_t)i);
            keys[i] = key;
            ids[i] = (uint32_t)i;
            hist.add(key);
        }
    }
    hist.finish_tile(blockIdx.x);
}

__global__ __launch_bounds__(kSmallBlock) void k_order_queries_small(QueryParams q, GridParams g, int bits,
                                                                     uint32_t *__restrict__ keys,
                                                                     uint32_t *__restrict__ order) {
    __shared__ SmallSortLds L;
    small_sort(L, (uint32_t)q.n, bits, [&](uint32_t i) { return query_key(q, g, i); }, keys, order);
}

// The queries of a quarter of a cell in spatial order, for the dense cells'
// walk: by place code, stably, inside blocks of kRefineTile consecutive
// queries of the plan, so that runs of queries with one code prefix lie in
// one box. Also their positions in that order, the code in the w component.
// Bound by the random reads of 12-byte positions, which the sampler used to
// make itself.
constexpr int kRefineItems = 4;
constexpr int kRefineTile = kBlock * kRefineItems;  // 1024
// The place of a query in its quarter of a cell, bits from the top: halves
// of the cell along z and y, quarters along z and y. A prefix of 2 bits names a
// box of 1/4 x 1/2 x 1/2 of the cell, all four a cube of side 1/4.
constexpr int kPlaceBits = 4;
// A block is left as it is when no run of one quarter is longer than this.
constexpr int kRefineRun = 16;

__device__ __forceinline__ uint32_t place_code(const GridParams &g, uint32_t key, float py, float pz) {
    const uint32_t cyz = key / kSub / (uint32_t)g.cells[0], ny = (uint32_t)g.cells[1];
    const uint32_t cz = cyz / ny, cy = cyz - cz * ny;
    const float ty = (py - g.lo[1]) * g.invc[1] - (float)cy, tz = (pz - g.lo[2]) * g.invc[2] - (float)cz;
    // quarters of the cell, 0..3
    const uint32_t iy = (uint32_t)fminf(fmaxf(ty * 4.0f, 0.0f), 3.0f);
    const uint32_t iz = (uint32_t)fminf(fmaxf(tz * 4.0f, 0.0f), 3.0f);
    return ((iz >> 1) << 3) | ((iy >> 1) << 2) | ((iz & 1u) << 1) | (iy & 1u);
}

// Stable places of the block's kRefineTile elements by digit (< 2^bits):
// element (wave, i, lane), in that order, gets slot[i]. cnt: kWavesPerBlock
// << bits words of LDS; waves rank their rows with one ballot per digit bit
// and a running count per digit, as the radix sort does.
__device__ __forceinline__ void block_split(const uint32_t (&d)[kRefineItems], int bits, uint32_t *cnt, uint32_t *scan,
                                            uint32_t (&slot)[kRefineItems]) {
    const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, nd = 1u << bits;
    for (uint32_t i = tid; i < kWavesPerBlock * nd; i += kBlock) cnt[i] = 0;
    __syncthreads();
    const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (64 - lane);
    uint32_t *mine = cnt + wave * nd;
#pragma unroll
    for (int i = 0; i < kRefineItems; ++i) {
        uint64_t m = ~0ull;
        for (int b = 0; b < bits; ++b) {
            const bool bit = (d[i] >> b) & 1u;
            const uint64_t bm = __ballot(bit);
            m &= bit ? bm : ~bm;
        }
        const uint32_t before = (uint32_t)__popcll(m & lt);
        const uint32_t base = mine[d[i]];
        // every lane of the wave has read the counter before its leader writes
        __builtin_amdgcn_wave_barrier();
        if (before == 0) mine[d[i]] = base + (uint32_t)__popcll(m);
        __builtin_amdgcn_wave_barrier();
        slot[i] = base + before;
    }
    __syncthreads();
    // exclusive scan over (digit, wave): thread t takes nd / kBlock digits
    const uint32_t per = (nd + kBlock - 1) / kBlock;
    uint32_t s = 0;
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t dg = tid * per + j;
        if (dg < nd)
            for (uint32_t w = 0; w < kWavesPerBlock; ++w) s += cnt[w * nd + dg];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan(s, scan, &tot);
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t dg = tid * per + j;
        if (dg < nd)
            for (uint32_t w = 0; w < kWavesPerBlock; ++w) {
                const uint32_t t = cnt[w * nd + dg];
                cnt[w * nd + dg] = run;
                run += t;
            }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRefineItems; ++i) slot[i] += mine[d[i]];
    __syncthreads();
}

__global__ __launch_bounds__(kBlock) void k_refine_order(QueryParams q, GridParams g,
                                                         const uint32_t *__restrict__ boxed,
                                                         const uint32_t *__restrict__ keys, uint32_t *order,
                                                         float4 *__restrict__ pos) {
    if (boxed[0] == 0) return;
    __shared__ float4 s_pos[kRefineTile];
    __shared__ uint32_t s_pid[kRefineTile];
    __shared__ uint32_t s_cnt[kWavesPerBlock * kRefineTile];  // up to kRefineTile runs
    __shared__ uint16_t s_run[kRefineTile], s_at[kRefineTile];
    __shared__ uint32_t s_scan[kWavesPerBlock];
    const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int64_t base = (int64_t)blockIdx.x * kRefineTile;
    const uint32_t have = q.n - base < kRefineTile ? (uint32_t)(q.n - base) : (uint32_t)kRefineTile;
    uint32_t pid[kRefineItems], code[kRefineItems], starts = 0;
    float4 p[kRefineItems];
    bool first[kRefineItems];
    bool longrun = false;
#pragma unroll
    for (int i = 0; i < kRefineItems; ++i) {
        const uint32_t e = wave * (kWave * kRefineItems) + (uint32_t)i * kWave + lane;
        pid[i] = 0;
        code[i] = 0;
        first[i] = false;
        p[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (e < have) {
            const uint32_t key = keys[base + e];
            pid[i] = order[base + e];
            first[i] = e == 0 || keys[base + e - 1] != key;
            longrun = longrun || (e + kRefineRun < have && keys[base + e + kRefineRun] == key);
            bool valid;
            query_position(q, g, pid[i], p[i].x, p[i].y, p[i].z, valid);
            if (key < kSub * (uint32_t)g.ncells) code[i] = place_code(g, key, p[i].y, p[i].z);
            p[i].w = __uint_as_float(code[i]);
        } else {
            first[i] = e == have;  // the elements past the end are a last run
        }
        starts += (uint32_t)__popcll(__ballot(first[i]));
    }
    if (__syncthreads_or(longrun) == 0) {
#pragma unroll
        for (int i = 0; i < kRefineItems; ++i) {
            const uint32_t e = wave * (kWave * kRefineItems) + (uint32_t)i * kWave + lane;
            if (e < have) {
                pos[base + e] = p[i];
            }
        }
        return;
    }
    // runs in order, then each by place: stable splits by place and by run
    if (lane == 0) s_scan[wave] = starts;
    __syncthreads();
    uint32_t run = 0, nruns = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)kWavesPerBlock; ++w) {
        if (w < wave) run += s_scan[w];
        nruns += s_scan[w];
    }
    __syncthreads();
    const uint64_t le = ~0ull >> (63 - lane);
#pragma unroll
    for (int i = 0; i < kRefineItems; ++i) {
        const uint32_t e = wave * (kWave * kRefineItems) + (uint32_t)i * kWave + lane;
        const uint64_t m = __ballot(first[i]);
        s_run[e] = (uint16_t)(run + (uint32_t)__popcll(m & le) - 1u);
        run += (uint32_t)__popcll(m);
        s_pos[e] = p[i];
        s_pid[e] = pid[i];
    }
    uint32_t slot[kRefineItems];
    block_split(code, kPlaceBits, s_cnt, s_scan, slot);
#pragma unroll
    for (int i = 0; i < kRefineItems; ++i)
        s_at[slot[i]] = (uint16_t)(wave * (kWave * kRefineItems) + (uint32_t)i * kWave + lane);
    __syncthreads();
    if (nruns > 1) {
        uint32_t d[kRefineItems], el[kRefineItems];
#pragma unroll
        for (int i = 0; i < kRefineItems; ++i) {
            el[i] = s_at[wave * (kWave * kRefineItems) + (uint32_t)i * kWave + lane];
            d[i] = s_run[el[i]];
        }
        block_split(d, 32 - __builtin_clz(nruns - 1u), s_cnt, s_scan, slot);
#pragma unroll
        for (int i = 0; i < kRefineItems; ++i) s_at[slot[i]] = (uint16_t)el[i];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kRefineItems; ++i) {
        const uint32_t e = (uint32_t)i * kBlock + tid;
        if (e < have) {
            const uint32_t at = s_at[e];
            order[base + e] = s_pid[at];
            pos[base + e] = s_pos[at];
        }
    }
}

// Work items of the ordered-query sampler: one per cell holding fewer than
// 2 kDenseMin queries, one per dense item (64 or 128 queries, see
// dense_item_queries) of a denser cell. The bucket of queries outside the
// domain (key ncells) is an item with an empty list.
constexpr uint32_t kDenseMin = 32;
// A cell of at least 2 kDenseMin queries is dense: lanes are its queries,
// one or two per lane, the cell's queries split evenly over its items. Two
// a lane let each record read from LDS serve two queries (with one, the
// walk is bound by LDS reads: three 16-byte broadcast reads per candidate
// against 13 VALU operations), but make half as many items, each twice as
// long: a launch with few items per wave slot of the chip then ends with
// long items running alone. Two a lane are taken from kDenseBalance items
// per wave slot at one a lane (measured, one and two a lane: 4.6 per slot, a
// 2^21-point batch of clustered points, 11 % faster with one; 33 per slot, 15 M
// points in 40^3 cells, 1.10 and 0.98 ms uniform, 2.99 and 2.47 clustered; 218
// per slot, 10^8 points in 64^3 cells, 11.3 and 11.5 uniform, 17.0 and 14.3
// clustered).
constexpr uint32_t kDenseBalance = 32;
// Queries of a boxed launch's dense items, each taken by a workgroup whose
// waves share the cell's records in LDS. Sixteen tiles, one pass of four
// waves with four tiles each, hold 256 queries when every tile is full; tiles
// do not cross boxes, so 192 fill them about as far as they go.
constexpr uint32_t kBoxedQ = 192;
constexpr uint32_t kChunkB = 8;  // queries evaluated together by a sparse-cell item
constexpr uint32_t kRowsMin = 4;                 // from this many queries a cell uses 4 query rows
constexpr uint32_t kRowsMax = (kDenseMin + 3) / 4;  // queries per row at most

// Work items per bucket (cell, and the outside bucket last): none for an
// empty bucket, one for a sparse one, one per dense_q queries of a dense
// one. Dense buckets' items come first in the item list, then the sparse
// buckets', each class in bucket order: items are taken in launch order,
// and the long ones started first leave no long item running alone at the
// end of the launch. The counts travel packed as (dense << 32) | sparse.
__device__ __forceinline__ uint64_t bucket_items(const uint32_t *point_off, int64_t c, int64_t nbuckets,
                                                 uint32_t dense_q) {
    if (c >= nbuckets) return 0ull;
    // the outside bucket (c = nbuckets - 1) has a single key
    const uint32_t n = point_off[c + 1 < nbuckets ? kSub * (c + 1) : kSub * c + 1] - point_off[kSub * c];
    if (n == 0) return 0ull;
    if (n < 2 * kDenseMin) return 1ull;
    return (uint64_t)((n + dense_q - 1) / dense_q) << 32;
}

// Buckets are taken kItemGroup at a time (kItemsPerThread per thread).
constexpr int kItemsPerThread = 4;
constexpr int kItemGroup = kBlock * kItemsPerThread;  // 1024
// Up to this many groups, the offsets kernel sums the other groups itself;
// beyond, their sums are scanned by a separate pass (which also writes the
// total after them).
constexpr int64_t kInlineGroups = 1024;

// With cell_off also the pairs the group's queries test (queries times list).
__global__ __launch_bounds__(kBlock) void k_item_sums(const uint32_t *__restrict__ point_off, int64_t nbuckets,
                                                      uint32_t dense_q, uint64_t *__restrict__ group_sum,
                                                      const uint32_t *__restrict__ cell_off,
                                                      uint64_t *__restrict__ group_vote) {
    __shared__ uint64_t lds[kWavesPerBlock];
    const int64_t base = (int64_t)blockIdx.x * kItemGroup + (int64_t)threadIdx.x * kItemsPerThread;
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < kItemsPerThread; ++i) s += bucket_items(point_off, base + i, nbuckets, dense_q);
    uint64_t tot;
    (void)block_excl_scan(s, lds, &tot);
    if (threadIdx.x == 0) group_sum[blockIdx.x] = tot;
    if (!cell_off) return;
    uint64_t p = 0;
#pragma unroll
    for (int i = 0; i < kItemsPerThread; ++i) {
        const int64_t c = base + i;
        if (c + 1 < nbuckets)
            p += (uint64_t)(point_off[kSub * (c + 1)] - point_off[kSub * c]) * (cell_off[c + 1] - cell_off[c]);
    }
    (void)block_excl_scan(p, lds, &tot);
    if (threadIdx.x == 0) group_vote[blockIdx.x] = tot;
}

// item_off[c] for c <= nbuckets: the first item of bucket c (item_off[nbuckets]
// = the total), and the item list: item_off[c] .. item_off[c] + items(c) - 1
// name bucket c. group_sum: the groups' sums, or (scanned) their exclusive
// prefixes followed by the total. With flags, the items of a launch that is
// boxed if its queries in the domain test `list` pairs or more on average
// (group_vote: as group_sum): flags[0] is then the dense items' number, else 0,
// without any items, and flags[1] 0.
__global__ __launch_bounds__(kBlock) void k_item_offsets(const uint32_t *__restrict__ point_off, int64_t nbuckets,
                                                         uint32_t dense_q, const uint64_t *__restrict__ group_sum,
                                                         int64_t ngroups,
                                                         bool scanned, uint32_t *__restrict__ item_off,
                                                         uint32_t *__restrict__ items, int64_t max_items,
                                                         const uint64_t *__restrict__ group_vote, uint32_t list,
                                                         uint32_t *__restrict__ flags) {
    __shared__ uint64_t lds[kWavesPerBlock];
    uint64_t prefix, total;
    if (scanned) {
        prefix = group_sum[blockIdx.x];
        total = group_sum[ngroups];
    } else {
        uint64_t p = 0, a = 0;
        for (uint32_t j = threadIdx.x; j < (uint32_t)ngroups; j += kBlock) {
            const uint64_t v = group_sum[j];
            a += v;
            if (j < blockIdx.x) p += v;
        }
        uint64_t t;
        (void)block_excl_scan(p, lds, &t);
        prefix = t;
        (void)block_excl_scan(a, lds, &t);
        total = t;
    }
    const uint32_t dense_total = (uint32_t)(total >> 32);
    if (flags) {
        uint64_t vote = 0;
        if (scanned) {
            vote = group_vote[ngroups];
        } else {
            for (uint32_t j = threadIdx.x; j < (uint32_t)ngroups; j += kBlock) vote += group_vote[j];
            uint64_t t;
            (void)block_excl_scan(vote, lds, &t);
            vote = t;
        }
        const bool boxed = vote >= (uint64_t)list * point_off[kSub * (nbuckets - 1)];
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            flags[0] = boxed ? dense_total : 0u;
            flags[1] = 0;
        }
        if (!boxed) return;
    }
    const int64_t base = (int64_t)blockIdx.x * kItemGroup + (int64_t)threadIdx.x * kItemsPerThread;
    uint64_t v[kItemsPerThread];
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < kItemsPerThread; ++i) {
        v[i] = bucket_items(point_off, base + i, nbuckets, dense_q);
        s += v[i];
    }
    uint64_t tot;
    uint64_t run = block_excl_scan(s, lds, &tot) + prefix;
#pragma unroll
    for (int i = 0; i < kItemsPerThread; ++i) {
        const int64_t c = base + i;
        const bool dense = (v[i] >> 32) != 0;
        const uint32_t first = dense ? (uint32_t)(run >> 32) : dense_total + (uint32_t)run;
        const uint32_t cnt = dense ? (uint32_t)(v[i] >> 32) : (uint32_t)v[i];
        if (c < nbuckets) item_off[c] = first;
        if (c == nbuckets) item_off[c] = dense_total + (uint32_t)total;
        for (uint32_t k = 0; k < cnt; ++k)
            if ((int64_t)(first + k) < max_items) items[first + k] = (uint32_t)c;
        run += v[i];
    }
}

// G of a record at a point, 0 past the cutoff.
__device__ __forceinline__ float eval_g(const Record &r, float px, float py, float pz, float T) {
    const float Q = cutoff_q(r, px, py, pz);
    return Q <= T ? exp2_hw(-Q) : 0.0f;
}

// sum over the 64 lanes, returned to every lane
__device__ __forceinline__ float wave_total(float x) {
    const float r = row16_sum(x);
    return (readlane_f(r, 0) + readlane_f(r, 16)) + (readlane_f(r, 32) + readlane_f(r, 48));
}

// Outputs of one query: (Phi, I) at its id in query order, and its position
// and (Phi, I) at its index k in plan order for the backward.
__device__ __forceinline__ void write_out(float I, float V, float tau, bool work, uint32_t pid, uint32_t k, float px,
                                          float py, float pz, float *out_v, float *out_i, const PlanResults &pr) {
    const bool def = work && I > tau;
    const float phi = def ? V / I : 0.0f, inf = def ? I : 0.0f;
    out_v[pid] = phi;
    out_i[pid] = inf;
    pr.pos[k] = make_float4(px, py, pz, 0.0f);
    pr.out[k] = make_float2(phi, inf);
}

// The same where the plan holds the positions already (boxed launches).
__device__ __forceinline__ void write_out(float I, float V, float tau, uint32_t pid, uint32_t k, float *out_v,
                                          float *out_i, float2 *plan_out) {
    const bool def = I > tau;
    const float phi = def ? V / I : 0.0f, inf = def ? I : 0.0f;
    out_v[pid] = phi;
    out_i[pid] = inf;
    plan_out[k] = make_float2(phi, inf);
}

// Sum over the SL lanes of a candidate-slot row (16: DPP row sum; 8: quad
// sums, then row_half_mirror pairs the two quads of each half row).
template <uint32_t SL>
__device__ __forceinline__ float slot_sum(float x) {
    if (SL == 16) return row16_sum(x);
    x += dpp_f<0xB1>(x);
    x += dpp_f<0x4E>(x);
    x += dpp_f<0x141>(x);
    return x;
}

// ROWS query rows x (64 / ROWS) candidate slots for a cell of
// n < 8 ROWS queries: lane (r, s) evaluates queries r, r + ROWS, ... against
// candidates s, s + 64 / ROWS, ... of the list; a query's partial sums are
// then summed over its row with DPP.
template <uint32_t ROWS>
__device__ __forceinline__ void query_rows(uint32_t lane, uint32_t n, uint32_t pa, uint32_t ja, uint32_t jb,
                                           uint32_t c, uint32_t ncells, const QueryParams &q, const GridParams &g,
                                           const Record *__restrict__ rec, const uint32_t *__restrict__ gids,
                                           const uint32_t *__restrict__ order, float T, float tau,
                                           float *__restrict__ out_v, float *__restrict__ out_i,
                                           const PlanResults &pr, float4 *buf) {
        constexpr uint32_t SL = kWave / ROWS;  // candidate slots per row
        const uint32_t row = lane / SL, sl = lane % SL;
        const uint32_t nt = (n + ROWS - 1) / ROWS;  // queries per row, <= kRowsMax
        uint32_t pid = 0;
        float mx = 0.0f, my = 0.0f, mz = 0.0f;
        bool valid = false;
        if (lane < n) {
            pid = order[pa + lane];
            if ((int64_t)pid < q.n) query_position(q, g, pid, mx, my, mz, valid);
        }
        float px[kRowsMax], py[kRowsMax], pz[kRowsMax], Ip[kRowsMax], Vp[kRowsMax];
#pragma unroll
        for (uint32_t t = 0; t < kRowsMax; ++t) {
            px[t] = py[t] = pz[t] = 0.0f;
            Ip[t] = Vp[t] = 0.0f;
            if (t < nt) {
                const int src = (int)(row + ROWS * t);
                px[t] = __shfl(mx, src, 64);
                py[t] = __shfl(my, src, 64);
                pz[t] = __shfl(mz, src, 64);
            }
        }
        // The list is taken 64 candidates at a time: lane l copies candidate
        // c0 + l's record from memory straight into the wave's LDS planes
        // (lanes past the list copy its last record), the ids of the next 64
        // are fetched meanwhile, and the steps of SL read the records from
        // LDS, so a chunk waits for memory once instead of once per step.
        uint32_t gnext = 0;
        if (ja < jb) gnext = gids[ja + lane < jb ? ja + lane : jb - 1];
        for (uint32_t c0 = ja; c0 < jb; c0 += kWave) {
            const float4 *src = (const float4 *)(rec + gnext);
#pragma unroll
            for (int qq = 0; qq < kRecordQuads; ++qq)
                __builtin_amdgcn_global_load_lds((const void *)(src + qq),
                                                 (__attribute__((address_space(3))) void *)(buf + qq * kWave), 16, 0, 0);
            if (c0 + kWave < jb) gnext = gids[c0 + kWave + lane < jb ? c0 + kWave + lane : jb - 1];
            __builtin_amdgcn_s_waitcnt(0);
            __builtin_amdgcn_wave_barrier();
            const uint32_t left = jb - c0;
            const uint32_t nstep = left >= (uint32_t)kWave ? kWave / SL : (left + SL - 1) / SL;
            for (uint32_t st = 0; st < nstep; ++st) {
                const uint32_t sidx = SL * st + sl;
                Record r;
                r.f0 = buf[sidx];
                r.f1 = buf[kWave + sidx];
                r.f2 = buf[2 * kWave + sidx];
                if (c0 + sidx >= jb) r.f0.w = r.f1.w = 0.0f;  // past the list: weight 0
#pragma unroll
                for (uint32_t t = 0; t < kRowsMax; ++t) {
                    if (t < nt) {
                        const float G = eval_g(r, px[t], py[t], pz[t], T);
                        Ip[t] = fmaf_(r.f0.w, G, Ip[t]);
                        Vp[t] = fmaf_(r.f1.w, G, Vp[t]);
                    }
                }
            }
            // every lane has read the planes before the next chunk overwrites them
            __builtin_amdgcn_wave_barrier();
        }
        float Io = 0.0f, Vo = 0.0f;
#pragma unroll
        for (uint32_t t = 0; t < kRowsMax; ++t) {
            if (t < nt) {
                const float It = slot_sum<SL>(Ip[t]), Vt = slot_sum<SL>(Vp[t]);
                if (sl == t) {
                    Io = It;
                    Vo = Vt;
                }
            }
        }
        // lane (r, t) writes query r + ROWS t, whose id and position that lane holds
        const uint32_t qi = row + ROWS * sl;
        const int src = (int)(qi & 63u);
        const uint32_t wpid = __shfl(pid, src, 64);
        const float wx = __shfl(mx, src, 64), wy = __shfl(my, src, 64), wz = __shfl(mz, src, 64);
        const bool wvalid = __shfl((int)valid, src, 64) != 0;
        if (sl < nt && qi < n && (int64_t)wpid < q.n)
            write_out(Io, Vo, tau, wvalid && c < ncells, wpid, pa + qi, wx, wy, wz, out_v, out_i, pr);
}

// A dense cell's work item: queries [qa, qa + qn) of the plan, qn <= 64 R;
// lane l takes queries qa + l + 64 t, t < R.
template <uint32_t R>
__device__ __forceinline__ void dense_item(uint32_t lane, uint32_t qa, uint32_t qn, uint32_t ja,
                                           uint32_t jb, uint32_t c, uint32_t ncells, const QueryParams &q,
                                           const GridParams &g, const Record *__restrict__ rec,
                                           bool off, const uint32_t *__restrict__ gids,
                                           const uint32_t *__restrict__ order, float T, float tau,
                                           float *__restrict__ out_v, float *__restrict__ out_i,
                                           const PlanResults &pr, float4 *buf) {
    float px[R], py[R], pz[R], I[R], V[R];
    uint32_t pid[R];
    bool valid[R];
#pragma unroll
    for (uint32_t t = 0; t < R; ++t) {
        px[t] = py[t] = pz[t] = 0.0f;
        I[t] = V[t] = 0.0f;
        pid[t] = 0xFFFFFFFFu;
        valid[t] = false;
        if (lane + kWave * t < qn) {
            pid[t] = order[qa + lane + kWave * t];
            if ((int64_t)pid[t] < q.n) query_position(q, g, pid[t], px[t], py[t], pz[t], valid[t]);
        }
    }
    float ox = 0.0f, oy = 0.0f, oz = 0.0f;
    if (c < ncells) cell_centre(g, c, ox, oy, oz);
    walk_staged_r<R>(rec, off, gids, ja, jb, lane, buf, px, py, pz, ox, oy, oz, T, I, V);
#pragma unroll
    for (uint32_t t = 0; t < R; ++t)
        if (lane + kWave * t < qn && (int64_t)pid[t] < q.n)
            write_out(I[t], V[t], tau, valid[t] && c < ncells, pid[t], qa + lane + kWave * t, px[t], py[t], pz[t],
                      out_v, out_i, pr);
}

// A boxed launch orders its queries by place too (k_refine_order) and cuts
// dense cells into boxes, prefixes of the place code (dense_level: how many of
// its bits; quarters of the cell along x at 0). A tile holds queries of one
// box, and meets only the candidates whose ellipsoid can reach the box. The
// more queries a cell has, the finer its boxes: each level tests about half
// the pairs of the one before, and a box should fill a tile; cells of fewer
// than kLevel2Queries are one box. The level depends on the cell's count only
// and the boxes on the grid, so a query's sums do not depend on how the
// queries were split into items.
// What the boxes save grows with the lists that the queries meet; what they
// cost, the order by place (22 to 28 ps a query) and the list tests, does not.
// So a launch is boxed when its queries test kBoxedList1 pairs or more on
// average, kBoxedList2 where the other walk has two queries a lane. The device
// decides (k_item_offsets), as the average list of a cell, which the host
// knows, says little: clustered queries meet lists of several times that. Only
// launches of kBoxedMean queries a cell and kBoxedQueries queries ask: below,
// cells would mostly be one box, and the longer items leave the chip idle at
// the end; and none whose cells list fewer than kVoteList pairs on average.
// Forward with its ordering, boxed over unboxed time, uniform and clustered
// points in 4^3 to 64^3 cells, by the pairs a query tests: 2 to 4 M queries
// 1.24 to 1.47 at 100 to 200, 0.84 to 1.16 at 240 to 310, 0.73 to 0.93 from 348;
// 4 to 8 M 1.13 to 1.64 at 89 to 220, 0.90 to 1.08 at 250 to 315, 0.62 to 1.02
// from 330; 8 to 14.7 M 1.19 to 1.48 to 177, 0.93 to 1.13 at 238 to 297, 0.63 to
// 0.94 from 325. 15 to 35 M (two a lane) 1.02 to 1.60 to 348, 0.96 to 1.13 at 450
// to 566, 0.60 to 1.00 from 725; 10^8 0.90 at 829. 1 to 2 M: 1.20 at 371, 0.74 to
// 1.02 from 489. Asking costs a launch that is not boxed some 15 us (4 M uniform
// points in 20^3 cells 335 -> 344 us; from 8 M less than the runs differ).
constexpr int64_t kBoxedMean = 320, kBoxedQueries = (int64_t)1 << 21, kVoteList = 60;
constexpr int64_t kBoxedList1 = 320, kBoxedList2 = 600;
constexpr uint32_t kLevel2Queries = (uint32_t)kBoxedMean, kLevel4Queries = 1536;
constexpr uint32_t kWholeCell = 32;  // no level: one box
__device__ __forceinline__ uint32_t dense_level(uint32_t n) {
    return n < kLevel2Queries ? kWholeCell : (n < kLevel4Queries ? 2u : 4u);
}

// A box of the cell about its centre: centre and half extents, the latter
// widened by slack (the queries' places are computed in float32).
struct Box3 {
    float cx, cy, cz, hx, hy, hz;
};

// bin: quarter along x, then `level` bits of the place code (z and y halves,
// z and y quarters).
__device__ __forceinline__ Box3 cell_box(uint32_t bin, uint32_t level, float wx, float wy, float wz,
                                         const float (&slack)[3]) {
    Box3 b;
    if (level == kWholeCell) {
        b.cx = b.cy = b.cz = 0.0f;
        b.hx = 0.5f * wx + slack[0];
        b.hy = 0.5f * wy + slack[1];
        b.hz = 0.5f * wz + slack[2];
        return b;
    }
    const uint32_t qx = bin >> level;
    uint32_t iz = 0, iy = 0;
    float parts = 1.0f;
    if (level == 2) {
        iz = (bin >> 1) & 1u;
        iy = bin & 1u;
        parts = 2.0f;
    } else if (level == 4) {
        iz = ((bin >> 3) & 1u) * 2u + ((bin >> 1) & 1u);
        iy = ((bin >> 2) & 1u) * 2u + (bin & 1u);
        parts = 4.0f;
    }
    b.hx = 0.125f * wx;
    b.hy = 0.5f * wy / parts;
    b.hz = 0.5f * wz / parts;
    b.cx = (2.0f * (float)qx + 1.0f) * b.hx - 0.5f * wx;
    b.cy = (2.0f * (float)iy + 1.0f) * b.hy - 0.5f * wy;
    b.cz = (2.0f * (float)iz + 1.0f) * b.hz - 0.5f * wz;
    b.hx += slack[0];
    b.hy += slack[1];
    b.hz += slack[2];
    return b;
}

// The staged candidates [0, cnt) whose ellipsoid may reach the box, in order,
// into the wave's list, padded with the all-zero record to whole tiles;
// returns their number. Each component of u over the box lies within
// |U_i| h of its value at the box's centre, so Q' is at least the sum of the
// squares that are left; Tm is the cutoff widened for the rounding of both.
__device__ __forceinline__ uint32_t list_reaching(DenseLds &L, uint32_t wave, uint32_t lane, uint32_t cnt,
                                                  const Box3 &x, float Tm) {
    uint16_t *list = L.list[wave];
    uint32_t S = 0;
    for (uint32_t c = 0; c < cnt; c += kWave) {
        const uint32_t j = c + lane;
        const float4 r0 = L.b[0][j], r1 = L.b[1][j], r2 = L.b[2][j];
        const float e0 = fmaf_(r0.w, x.cx, fmaf_(r0.z, x.cy, fmaf_(r0.y, x.cz, r0.x)));
        const float e1 = fmaf_(r1.z, x.cy, fmaf_(r1.y, x.cz, r1.x));
        const float e2 = fmaf_(r2.y, x.cz, r2.x);
        const float h0 = fmaf_(fabsf(r0.w), x.hx, fmaf_(fabsf(r0.z), x.hy, fabsf(r0.y) * x.hz));
        const float h1 = fmaf_(fabsf(r1.z), x.hy, fabsf(r1.y) * x.hz);
        const float h2 = fabsf(r2.y) * x.hz;
        const float d0 = fmaxf(fabsf(e0) - h0, 0.0f), d1 = fmaxf(fabsf(e1) - h1, 0.0f);
        const float d2 = fmaxf(fabsf(e2) - h2, 0.0f);
        const bool in = j < cnt && !(fmaf_(d0, d0, fmaf_(d1, d1, d2 * d2)) > Tm);
        const uint64_t m = __ballot(in);
        if (in) {
            const uint32_t at =
                S + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const float2 w = L.w[j];
            list[at] = (uint16_t)j;
            L.lw[wave][at] = w.x;
            L.lv[wave][at] = w.y;
        }
        S += (uint32_t)__popcll(m);
    }
    if (lane < kTile) {
        list[S + lane] = (uint16_t)kBlock;
        L.lw[wave][S + lane] = L.lv[wave][S + lane] = 0.0f;
    }
    __builtin_amdgcn_wave_barrier();
    return S;
}

// A dense cell's work item of a boxed launch: queries [qa, qa + qn) of the
// plan, qn <= kBoxedQ, by the whole workgroup. The queries are cut into tiles
// of up to 16 that do not cross a box (found with ballots over the queries'
// bins), at most kSlots of them to a wave and pass. The cell's records are staged kBlock at
// a time; each wave lists the ones that reach its tiles' box, and takes the
// list 16 candidates at a time.
constexpr uint32_t kSlots = 4;
__device__ __forceinline__ void dense_item(DenseLds &L, uint32_t wave, uint32_t lane, uint32_t qa, uint32_t qn,
                                           uint32_t n, uint32_t ja, uint32_t jb, uint32_t c, const GridParams &g,
                                           const Record *__restrict__ rec, const uint32_t *__restrict__ gids,
                                           const uint32_t *__restrict__ keys, const uint32_t *__restrict__ order,
                                           const float4 *__restrict__ pos, float T, float tau,
                                           float *__restrict__ out_v, float *__restrict__ out_i,
                                           float2 *__restrict__ plan_out) {
    const uint32_t tid = threadIdx.x, level = dense_level(n);
    float ox, oy, oz;
    cell_centre(g, c, ox, oy, oz);
    const float wx = 1.0f / g.invc[0], wy = 1.0f / g.invc[1], wz = 1.0f / g.invc[2];
    const float slack[3] = {0x1p-19f * (fabsf(g.lo[0]) + fabsf(g.hi[0]) + wx),
                            0x1p-19f * (fabsf(g.lo[1]) + fabsf(g.hi[1]) + wy),
                            0x1p-19f * (fabsf(g.lo[2]) + fabsf(g.hi[2]) + wz)};
    const float Tm = T * (1.0f + 0x1p-14f);
    // tiles: a query starts one at the start of its run of one bin, and 16,
    // 32, ... queries into it
    uint32_t bin = 0;
    bool start = false;
    if (level == kWholeCell) {
        start = tid == 0;
    } else if (tid < qn) {
        const uint32_t shift = (uint32_t)kPlaceBits - level;
        auto bin_at = [&](uint32_t k) {
            return ((keys[k] % kSub) << level) | (__float_as_uint(pos[k].w) >> shift);
        };
        bin = bin_at(qa + tid);
        start = tid == 0 || bin_at(qa + tid - 1) != bin;
    }
    const uint64_t le = ~0ull >> (63 - lane);
    const uint64_t sm = __ballot(start);
    if (lane == 0) L.ballot[0][wave] = sm;
    __syncthreads();
    uint32_t rs = 0;  // start of the query's run
    for (uint32_t w = 0; w <= wave; ++w) {
        const uint64_t m = w == wave ? (sm & le) : L.ballot[0][w];
        if (m != 0) rs = kWave * w + 63u - (uint32_t)__builtin_clzll(m);
    }
    const bool head = tid < qn && ((tid - rs) % kTile) == 0;
    const uint64_t hm = __ballot(head);
    if (lane == 0) L.ballot[1][wave] = hm;
    __syncthreads();
    uint32_t before = 0, nt = 0;
    for (uint32_t w = 0; w < (uint32_t)kDenseWaves; ++w) {
        const uint32_t cnt = (uint32_t)__popcll(L.ballot[1][w]);
        if (w < wave) before += cnt;
        nt += cnt;
    }
    if (head) {
        const uint32_t t = before + (uint32_t)__popcll(hm & le) - 1u;
        L.tile_start[t] = (uint16_t)tid;
        L.tile_bin[t] = (uint16_t)bin;
    }
    __syncthreads();
    const uint32_t k = lane >> 4;
    const uint32_t npass = (nt + kSlots * kDenseWaves - 1) / (kSlots * kDenseWaves);
    const uint32_t per = (nt + npass - 1) / npass;
    for (uint32_t pass = 0; pass < npass; ++pass) {
        const uint32_t t0 = pass * per, tn = nt - t0 < per ? nt - t0 : per;
        const uint32_t ta = t0 + tn * wave / kDenseWaves, tb = t0 + tn * (wave + 1) / kDenseWaves;
        float qt[kSlots], I[kSlots], V[kSlots];
        uint32_t ts[kSlots], tc[kSlots], tbin[kSlots];
#pragma unroll
        for (uint32_t t = 0; t < kSlots; ++t) {
            ts[t] = tc[t] = 0;
            tbin[t] = 0xFFFFFFFFu;
            qt[t] = I[t] = V[t] = 0.0f;
            if (ta + t < tb) {
                ts[t] = __builtin_amdgcn_readfirstlane(L.tile_start[ta + t]);
                tbin[t] = __builtin_amdgcn_readfirstlane(L.tile_bin[ta + t]);
                const uint32_t end =
                    ta + t + 1 < nt ? __builtin_amdgcn_readfirstlane(L.tile_start[ta + t + 1]) : qn;
                tc[t] = end - ts[t];
                // lanes past the tile's last query take that query again
                const uint32_t i = (lane & 15u) < tc[t] ? (lane & 15u) : tc[t] - 1u;
                const float4 p = pos[qa + ts[t] + i];
                qt[t] = tile_operand(k, p.x - ox, p.y - oy, p.z - oz);
            }
        }
        Record r = {};
        if (ja + tid < jb) r = load_record(rec, gids[ja + tid]);
        for (uint32_t c0 = ja; c0 < jb; c0 += kBlock) {
            __syncthreads();  // every wave has read the chunk before
            stage_rows(&L.b[0][tid], kBlock + 1, c0 + tid < jb, r, ox, oy, oz);
            L.w[tid] = make_float2(r.f0.w, r.f1.w);
            const uint32_t cn = c0 + kBlock;
            if (cn + tid < jb) r = load_record(rec, gids[cn + tid]);
            __syncthreads();
            const uint32_t cnt = jb - c0 < (uint32_t)kBlock ? jb - c0 : (uint32_t)kBlock;
            uint32_t S = 0;
#pragma unroll
            for (uint32_t t = 0; t < kSlots; ++t) {
                if (tbin[t] == 0xFFFFFFFFu) continue;
                if (t == 0 || tbin[t] != tbin[t - 1])
                    S = list_reaching(L, wave, lane, cnt, cell_box(tbin[t], level, wx, wy, wz, slack), Tm);
                const uint16_t *list = L.list[wave] + (lane & 15u);
                const float *lw = L.lw[wave] + 4u * k, *lv = L.lv[wave] + 4u * k;
                for (uint32_t s = 0; s < S; s += kTile) {
                    const float *p = (const float *)&L.b[0][list[s]] + k;
                    constexpr uint32_t plane = 4u * (kBlock + 1);
                    tile_pairs(qt[t], p[0], p[plane], p[2 * plane], *(const float4 *)(lw + s),
                               *(const float4 *)(lv + s), T, I[t], V[t]);
                }
            }
        }
        // lane l writes query l % 16 of tile l / 16
        static_assert(kSlots == 4, "a tile for every row of 16 lanes");
        const float Io = tile_sum(I[0], I[1], I[2], I[3]), Vo = tile_sum(V[0], V[1], V[2], V[3]);
        const uint32_t qs = k == 0 ? ts[0] : (k == 1 ? ts[1] : (k == 2 ? ts[2] : ts[3]));
        const uint32_t qc = k == 0 ? tc[0] : (k == 1 ? tc[1] : (k == 2 ? tc[2] : tc[3]));
        const uint32_t i = lane & 15u;
        if (i < qc) write_out(Io, Vo, tau, order[qa + qs + i], qa + qs + i, out_v, out_i, plan_out);
    }
}

// The dense items of a boxed launch: workgroups that fill the chip take two at
// a time (a cell's items follow one another) until none is left. (So a launch
// that turns out not to be boxed costs the workgroups that look and leave, not
// one for every item.)
constexpr uint32_t kDenseTake = 2;
__global__ __launch_bounds__(kBlock, kDensePerSimd) void k_sample_dense(
    GridParams g, const Record *__restrict__ rec, const uint8_t *__restrict__ cell_coarse,
    const uint32_t *__restrict__ gids, const uint32_t *__restrict__ cell_off, const uint32_t *__restrict__ point_off,
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ order, const uint32_t *__restrict__ item_off,
    const uint32_t *__restrict__ items, uint32_t *flags, float T, float tau, float *__restrict__ out_v,
    float *__restrict__ out_i, const float4 *__restrict__ pos, float2 *__restrict__ plan_out) {
    __shared__ DenseLds L;
    const uint32_t tid = threadIdx.x, lane = tid % kWave;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t ncells = (uint32_t)g.ncells;
    const uint32_t total = __builtin_amdgcn_readfirstlane(flags[0]);
    if (total == 0) return;
    for (;;) {
        if (tid == 0) {
            L.next = atomicAdd(flags + 1, kDenseTake);
            // the record that pads the lists (a coarse cell's records may lie on it)
            L.b[0][kBlock] = L.b[1][kBlock] = L.b[2][kBlock] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        __syncthreads();
        const uint32_t w0 = __builtin_amdgcn_readfirstlane(L.next);
        if (w0 >= total) return;
        for (uint32_t w = w0; w < w0 + kDenseTake && w < total; ++w) {
            const uint32_t c = ((ConstU32 *)items)[w], chunk = w - ((ConstU32 *)item_off)[c];
            const uint32_t pa = ((ConstU32 *)point_off)[kSub * c];
            const uint32_t n = ((ConstU32 *)point_off)[c < ncells ? kSub * (c + 1) : kSub * c + 1] - pa;
            uint32_t ja = 0, jb = 0;
            bool coarse = false;
            if (c < ncells) {
                ja = ((ConstU32 *)cell_off)[c];
                jb = ((ConstU32 *)cell_off)[c + 1];
                coarse = __builtin_amdgcn_readfirstlane(cell_coarse[c]) != 0;
            }
            const uint32_t nit = (n + kBoxedQ - 1) / kBoxedQ, per = (n + nit - 1) / nit;
            const uint32_t qa = pa + chunk * per, left = pa + n - qa, qn = left < per ? left : per;
            if (!coarse && ja < jb) {
                dense_item(L, wave, lane, qa, qn, n, ja, jb, c, g, rec, gids, keys, order, pos, T, tau, out_v, out_i,
                           plan_out);
            } else {
                // lanes are queries (an empty list leaves their sums at 0)
                float4 p = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (tid < qn) p = pos[qa + tid];
                float I = 0.0f, V = 0.0f;
                if (kWave * wave < qn)
                    walk_staged(rec, gids, ja, jb, lane, wave_records(L, wave), p.x, p.y, p.z, T, I, V);
                if (tid < qn) write_out(I, V, tau, order[qa + tid], qa + tid, out_v, out_i, plan_out);
            }
            __syncthreads();  // every wave is done with the item's LDS
        }
    }
}

// One wavefront per item, by the queries n of the cell:
//  * n >= 64: lanes are queries, up to dense_q / 64 each (dense_q
//    queries per item, a cell's queries split evenly over its items), and
//    walk the list together, the records staged in LDS;
//  * 4 <= n < 64: query rows x candidate slots (4 x 16 below 32 queries,
//    8 x 8 from 32), records staged in LDS 64 at a time;
//  * n < 4: lanes are the cell's candidates (64 at a time) and the queries
//    are visited in turn, their positions broadcast from SGPRs.
// Every query's sums are reduced in a fixed order.
// Seven waves per SIMD (at most 72 VGPRs, which the row layouts' per-row
// arrays need; eight would spill them to scratch).
__global__ __launch_bounds__(kSampBlock, kSampPerSimd) void k_sample_cells(QueryParams q, GridParams g, const Record *__restrict__ rec,
                                                         const uint8_t *__restrict__ cell_coarse,
                                                         const uint32_t *__restrict__ gids,
                                                         const uint32_t *__restrict__ cell_off,
                                                         const uint32_t *__restrict__ point_off,
                                                         const uint32_t *__restrict__ order,
                                                         const uint32_t *__restrict__ item_off,
                                                         const uint32_t *__restrict__ items, int64_t max_items,
                                                         uint32_t dense_q, const uint32_t *__restrict__ boxed_off,
                                                         const uint32_t *__restrict__ boxed_items,
                                                         const uint32_t *__restrict__ boxed_flags, float T, float tau,
                                                         float *__restrict__ out_v, float *__restrict__ out_i,
                                                         PlanResults pr) {
    // per wave: the records of 64 candidates, as three 1 KiB planes of
    // 16-byte quarters (quarter q of candidate s at [q][s])
    __shared__ float4 s_rec[kSampWaves][kRecordQuads * kWave];
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t ncells = (uint32_t)g.ncells;
    const uint32_t bid = xcd_group<kXcdItems>(blockIdx.x, gridDim.x);
    // a boxed launch has its own items; the dense ones, the first of the list,
    // are k_sample_dense's
    const uint32_t dense = boxed_flags ? ((ConstU32 *)boxed_flags)[0] : 0u;
    if (dense > 0) {
        item_off = boxed_off;
        items = boxed_items;
    }
    const uint64_t w = (uint64_t)bid * kSampWaves + threadIdx.x / kWave + dense;
    const uint32_t tot = ((ConstU32 *)item_off)[ncells + 1];
    const uint64_t total = tot < (uint64_t)max_items ? tot : (uint64_t)max_items;
    if (w >= total) return;
    const uint32_t c = __builtin_amdgcn_readfirstlane(((ConstU32 *)items)[w]);
    const uint32_t chunk = (uint32_t)w - ((ConstU32 *)item_off)[c];
    const uint32_t pa = ((ConstU32 *)point_off)[kSub * c];
    const uint32_t pb = ((ConstU32 *)point_off)[c < ncells ? kSub * (c + 1) : kSub * c + 1];
    const uint32_t n = pb - pa;
    uint32_t ja = 0, jb = 0;
    if (c < ncells) {
        ja = ((ConstU32 *)cell_off)[c];
        jb = ((ConstU32 *)cell_off)[c + 1];
    }
    if (n >= 2 * kDenseMin) {
        // offsets from the cell's centre unless the cell may list a Gaussian
        // too small for them (see offset_planes)
        const bool off = c >= ncells || __builtin_amdgcn_readfirstlane(cell_coarse[c]) == 0;
        const uint32_t nit = (n + dense_q - 1) / dense_q;
        const uint32_t per = (n + nit - 1) / nit;
        const uint32_t qa = pa + chunk * per;
        const uint32_t qn = pb - qa < per ? pb - qa : per;
        float4 *buf = s_rec[threadIdx.x / kWave];
        if (qn <= (uint32_t)kWave)
            dense_item<1>(lane, qa, qn, ja, jb, c, ncells, q, g, rec, off, gids, order, T, tau, out_v, out_i, pr,
                          buf);
        else
            dense_item<2>(lane, qa, qn, ja, jb, c, ncells, q, g, rec, off, gids, order, T, tau, out_v, out_i, pr,
                          buf);
        return;
    }
    if (n >= kRowsMin) {
        float4 *buf = s_rec[threadIdx.x / kWave];
        if (n >= kDenseMin)
            query_rows<8>(lane, n, pa, ja, jb, c, ncells, q, g, rec, gids, order, T, tau, out_v, out_i, pr, buf);
        else
            query_rows<4>(lane, n, pa, ja, jb, c, ncells, q, g, rec, gids, order, T, tau, out_v, out_i, pr, buf);
        return;
    }
    for (uint32_t p0 = pa; p0 < pb; p0 += kChunkB) {
        const uint32_t m = (pb - p0) < kChunkB ? (pb - p0) : kChunkB;
        uint32_t pid = 0;
        float mx = 0.0f, my = 0.0f, mz = 0.0f;
        bool valid = false;
        if (lane < m) {
            pid = order[p0 + lane];
            if ((int64_t)pid < q.n) query_position(q, g, pid, mx, my, mz, valid);
        }
        float Ip[kChunkB], Vp[kChunkB];
#pragma unroll
        for (uint32_t t = 0; t < kChunkB; ++t) Ip[t] = Vp[t] = 0.0f;
        for (uint32_t j0 = ja; j0 < jb; j0 += kWave) {
            const uint32_t j = j0 + lane;
            Record r;
            if (j < jb) {
                r = rec[gids[j]];
            } else {
                r.f0 = r.f1 = r.f2 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (uint32_t t = 0; t < kChunkB; ++t) {
                if (t < m) {
                    const float G = eval_g(r, readlane_f(mx, t), readlane_f(my, t), readlane_f(mz, t), T);
                    Ip[t] = fmaf_(r.f0.w, G, Ip[t]);
                    Vp[t] = fmaf_(r.f1.w, G, Vp[t]);
                }
            }
        }
        float Io = 0.0f, Vo = 0.0f;
#pragma unroll
        for (uint32_t t = 0; t < kChunkB; ++t) {
            if (t < m) {
                const float It = wave_total(Ip[t]), Vt = wave_total(Vp[t]);
                if (lane == t) {
                    Io = It;
                    Vo = Vt;
                }
            }
        }
        if (lane < m && (int64_t)pid < q.n)
            write_out(Io, Vo, tau, valid && c < ncells, pid, p0 + lane, mx, my, mz, out_v, out_i, pr);
    }
}

// Pairs the forward tests and the pairs among them that pass the cutoff,
// for measurement: thread t takes query t of the grid (x fastest) or the
// t-th query in plan order, walks its cell's list with the samplers' own
// float32 test and counts. Summed per block, then into totals[0] (tests)
// and totals[1] (passing) with one integer atomic each per block (the sums
// do not depend on their order).
__global__ __launch_bounds__(kBlock) void k_count_sample_pairs(QueryParams q, GridParams g,
                                                               const Record *__restrict__ rec,
                                                               const uint32_t *__restrict__ gids,
                                                               const uint32_t *__restrict__ cell_off,
                                                               const uint32_t *__restrict__ plan_keys,
                                                               const float4 *__restrict__ plan_pos, float T,
                                                               unsigned long long *totals) {
    __shared__ unsigned long long lds[2][kWavesPerBlock];
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    unsigned long long tests = 0, hits = 0;
    if (t < q.n) {
        int64_t c = -1;
        float px = 0.0f, py = 0.0f, pz = 0.0f;
        if (q.kind == 0) {
            const uint32_t nx = (uint32_t)q.dims[0], ny = (uint32_t)q.dims[1];
            const uint32_t vx = (uint32_t)(t % nx), vy = (uint32_t)((t / nx) % ny), vz = (uint32_t)(t / ((int64_t)nx * ny));
            const uint32_t rx = nx / (uint32_t)g.cells[0], ry = ny / (uint32_t)g.cells[1];
            const uint32_t rz = (uint32_t)q.dims[2] / (uint32_t)g.cells[2];
            c = (int64_t)(vx / rx) + (int64_t)g.cells[0] * ((int64_t)(vy / ry) + (int64_t)g.cells[1] * (vz / rz));
            px = voxel_center((int32_t)vx, g.lo[0], q.vsz[0]);
            py = voxel_center((int32_t)vy, g.lo[1], q.vsz[1]);
            pz = voxel_center((int32_t)vz, g.lo[2], q.vsz[2]);
        } else {
            const uint32_t cc = plan_keys[t] / kSub;
            if ((int64_t)cc < g.ncells) {
                c = cc;
                const float4 p = plan_pos[t];
                px = p.x;
                py = p.y;
                pz = p.z;
            }
        }
        if (c >= 0) {
            const uint32_t j0 = cell_off[c], j1 = cell_off[c + 1];
            tests = j1 - j0;
            for (uint32_t j = j0; j < j1; ++j) hits += cutoff_q(rec[gids[j]], px, py, pz) <= T ? 1u : 0u;
        }
    }
    const uint32_t lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        tests += __shfl_xor(tests, o, kWave);
        hits += __shfl_xor(hits, o, kWave);
    }
    if (lane == 0) {
        lds[0][wid] = tests;
        lds[1][wid] = hits;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long s = 0;
        for (int w = 0; w < kWavesPerBlock; ++w) s += lds[threadIdx.x][w];
        if (s) atomicAdd(totals + threadIdx.x, s);
    }
}

}  // namespace

hipError_t launch_count_sample_pairs(const QueryParams &q, const GridParams &g, const Record *rec,
                                     const uint32_t *gids, const uint32_t *cell_off, const uint32_t *plan_keys,
                                     const float4 *plan_pos, float T, unsigned long long *totals, hipStream_t s) {
    hipError_t e = fill_u32((uint32_t *)totals, 0u, 4, s);
    if (e != hipSuccess || q.n <= 0) return e;
    hipLaunchKernelGGL(k_count_sample_pairs, dim3((uint32_t)((q.n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, q, g,
                       rec, gids, cell_off, plan_keys, plan_pos, T, totals);
    return hipGetLastError();
}

hipError_t launch_order_queries_small(const QueryParams &q, const GridParams &g, int bits, uint32_t *keys,
                                      uint32_t *order, hipStream_t s) {
    if (q.n <= 0) return hipSuccess;
    prof_begin("order_small", s);
    hipLaunchKernelGGL(k_order_queries_small, dim3(1), dim3(kSmallBlock), 0, s, q, g, bits, keys, order);
    prof_end("order_small", s);
    return hipGetLastError();
}

hipError_t launch_query_keys(const QueryParams &q, const GridParams &g, uint32_t *keys, uint32_t *ids,
                             const RadixPass0 &pass0, hipStream_t s) {
    if (q.n <= 0) return hipSuccess;
    prof_begin("query_keys", s);
    hipLaunchKernelGGL(k_query_keys, dim3((uint32_t)((q.n + kSortTile - 1) / kSortTile)), dim3(kBlock), 0, s, q, g,
                       keys, ids, pass0);
    prof_end("query_keys", s);
    return hipGetLastError();
}

hipError_t launch_sample_grid(const QueryParams &q, const GridParams &g, const Record *rec, const uint32_t *gids,
                              const uint32_t *cell_off, float T, float tau, float *out_v, float *out_i,
                              hipStream_t s) {
    const int64_t vpc = (int64_t)(q.dims[0] / g.cells[0]) * (q.dims[1] / g.cells[1]) * (q.dims[2] / g.cells[2]);
    const int64_t wpc = (vpc + kWave - 1) / kWave;
    const int64_t blocks = g.ncells * wpc;
    if (blocks <= 0) return hipSuccess;
    // as many voxels a wave as the cell has, the list split over the lanes left
    const auto kernel = vpc > 64   ? k_sample_grid<1, 1>
                        : vpc > 48 ? k_sample_grid<4, 4>
                        : vpc > 32 ? k_sample_grid<4, 3>
                        : vpc > 16 ? k_sample_grid<4, 2>
                        : vpc > 8  ? k_sample_grid<4, 1>
                        : vpc > 4  ? k_sample_grid<8, 1>
                        : vpc > 1  ? k_sample_grid<16, 1>
                                   : k_sample_grid<64, 1>;
    prof_begin("sample_grid", s);
    hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), dim3(kWave), 0, s, q, g, rec, gids, cell_off, T,
                       tau, out_v, out_i);
    prof_end("sample_grid", s);
    return hipGetLastError();
}

static int compute_units() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
        (void)hipGetLastError();
        cus = 256;
    }
    return cus;
}

// Queries per dense work item for nq ordered queries on the current device:
// 128 (two a lane) from kDenseBalance items per wave slot of the chip at 64,
// else 64. The item list and the sampler both take it from nq, so they agree.
static uint32_t dense_item_queries(int64_t nq) {
    const int64_t slots = (int64_t)compute_units() * 4 * kSampPerSimd;  // 4 SIMDs a CU
    return nq / kWave >= (int64_t)kDenseBalance * slots ? 2u * kWave : (uint32_t)kWave;
}

int64_t boxed_list(int64_t nq, int64_t ncells, int64_t n_pairs) {
    if (nq < kBoxedMean * ncells || nq < kBoxedQueries || n_pairs < kVoteList * ncells) return -1;
    return dense_item_queries(nq) == (uint32_t)kWave ? kBoxedList1 : kBoxedList2;
}

// The items of buckets of `dense_q` queries an item, into item_off and items;
// with cell_off those of a boxed launch, if it is one.
static hipError_t list_items(const GridParams &g, const uint32_t *point_off, uint32_t dense_q, const PointItems &it,
                             uint32_t *item_off, uint32_t *items, int64_t max_items, const uint32_t *cell_off,
                             uint64_t *group_vote, uint32_t list, uint32_t *flags, hipStream_t s) {
    const int64_t nbuckets = g.ncells + 1;  // cells and the outside bucket
    // buckets 0..nbuckets-1 and one empty element after them (its offset is the total)
    const int64_t ngroups = (nbuckets + 1 + kItemGroup - 1) / kItemGroup;
    const bool scanned = ngroups > kInlineGroups;
    prof_begin("cell_items", s);
    hipLaunchKernelGGL(k_item_sums, dim3((uint32_t)ngroups), dim3(kBlock), 0, s, point_off, nbuckets, dense_q,
                       it.group_sum, cell_off, group_vote);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && scanned)
        e = exclusive_scan_u64_total(it.group_sum, it.group_sum, ngroups, it.group_sum + ngroups, it.scan_work, s);
    if (e == hipSuccess && scanned && group_vote)
        e = exclusive_scan_u64_total(group_vote, group_vote, ngroups, group_vote + ngroups, it.scan_work, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_item_offsets, dim3((uint32_t)ngroups), dim3(kBlock), 0, s, point_off, nbuckets,
                           dense_q, it.group_sum, ngroups, scanned, item_off, items, max_items, group_vote, list,
                           flags);
        e = hipGetLastError();
    }
    prof_end("cell_items", s);
    return e;
}

hipError_t launch_cell_items(int64_t nq, const GridParams &g, const uint32_t *point_off, const PointItems &it,
                             hipStream_t s) {
    if (nq <= 0) return hipSuccess;
    return list_items(g, point_off, dense_item_queries(nq), it, it.item_off, it.items, it.max_items, nullptr, nullptr,
                      0, nullptr, s);
}

hipError_t launch_boxed_items(const QueryParams &q, const GridParams &g, const uint32_t *cell_off,
                              const uint32_t *keys, const uint32_t *point_off, int64_t list, const PointItems &it,
                              const BoxedItems &b, uint32_t *order, float4 *pos, hipStream_t s) {
    hipError_t e = list_items(g, point_off, kBoxedQ, it, b.item_off, b.items, b.max_items, cell_off, b.group_vote,
                              (uint32_t)list, b.flags, s);
    if (e != hipSuccess) return e;
    prof_begin("refine_order", s);
    hipLaunchKernelGGL(k_refine_order, dim3((uint32_t)((q.n + kRefineTile - 1) / kRefineTile)), dim3(kBlock), 0, s, q,
                       g, b.flags, keys, order, pos);
    prof_end("refine_order", s);
    return hipGetLastError();
}

hipError_t launch_sample_points(const QueryParams &q, const GridParams &g, const Record *rec,
                                const uint8_t *cell_coarse, const uint32_t *gids, const uint32_t *cell_off,
                                const uint32_t *keys, const uint32_t *order, const uint32_t *point_off,
                                const PointItems &it, const BoxedItems &b, float T, float tau, float *out_v,
                                float *out_i, const PlanResults &pr, hipStream_t s) {
    if (q.n <= 0) return hipSuccess;
    prof_begin("sample_points", s);
    if (b.item_off) {
        hipLaunchKernelGGL(k_sample_dense, dim3((uint32_t)(compute_units() * kDensePerSimd)), dim3(kBlock), 0, s, g,
                           rec, cell_coarse, gids, cell_off, point_off, keys, order, b.item_off, b.items, b.flags, T,
                           tau, out_v, out_i, pr.pos, pr.out);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_sample_cells, dim3((uint32_t)((it.max_items + kSampWaves - 1) / kSampWaves)),
                       dim3(kSampBlock), 0, s, q, g, rec, cell_coarse, gids, cell_off, point_off, order, it.item_off,
                       it.items, it.max_items, dense_item_queries(q.n), b.item_off, b.items, b.flags, T, tau, out_v,
                       out_i, pr);
    prof_end("sample_points", s);
    return hipGetLastError();
}

}  // namespace gs
