// Ray-driven kernels: one thread per ray, walking its samples along k, with the sampled image staged
// in LDS (whole image, or row bands for large n).
//
//   k_att     attenuation scan, Eq. (1) inner integral: m = W mu, L_k = dx (m_k/2 + sum_{k'>k} m_k'),
//             att = exp(-L), scanned from the detector end with a compensated running sum, stored
//             no smaller than the smallest normal float (the paired kernels take its reciprocal).
//   k_fwd     attenuated projection, Eq. (2): y = dx sum_k att (W f), compensated; epilogues give the
//             MLEM ratio S/y or the Poisson NLL terms of Eq. (5).
//   k_fwd_pair  the same for two candidates per workgroup, sharing each sample's geometry.
//   k_adj_sweep  one reverse MLEM step along every ray: the projection adjoint of the ratio and the
//             attenuation adjoint accumulation, in one sweep.
//   k_tail    sensitivity adjoint, att = exp(-L) and the scan's transpose (a prefix sum).
//
// Layout: att and its adjoint are per-angle slabs in 4 x 8 (sample x bin) blocks (att_row / att_col
// in device_common.h). The threads of a wave take consecutive bins of one angle, so at each k a
// wave's loads cover whole 32-byte block rows, and a ray's offset splits into a per-lane bin part and
// a uniform sample-row part.
#include <type_traits>

#include "launch.h"

namespace boac {

// Map a flat workgroup id to (candidate, chunk) so that all chunks of one candidate run on the same
// XCD (workgroups are dispatched round-robin over the 8 XCDs); they share the candidate's image in L2.
__device__ __forceinline__ void ray_block(int bid, int chunks, int C, int &cand, int &chunk) {
    const int total = chunks * C;
    int id = bid;
    if ((total & 7) == 0) id = (id & 7) * (total >> 3) + (id >> 3);
    cand = id / chunks;
    chunk = id - cand * chunks;
}

constexpr int kMaxRpt = 4;
constexpr int kBandChunk = 16;  // samples per load batch in the row-band paths
constexpr int kRayChunk = 16;   // samples per load batch of the single-stage paths, in groups of 4
constexpr int kRayGroups = kRayChunk / 4;
__device__ __forceinline__ int ray_group(const DevGeom &g, int k0, int q) { return min(k0 + 4 * q, (g.nt - 1) & ~3); }

// A ray's running sum by a run-time index: selects, so that the sums stay in registers.
template <int N>
__device__ __forceinline__ Comp comp_pick(const Comp (&v)[N], int j) {
    Comp c = v[0];
#pragma unroll
    for (int i = 1; i < N; ++i) {
        c.s = (i == j) ? v[i].s : c.s;
        c.e = (i == j) ? v[i].e : c.e;
    }
    return c;
}
template <int N>
__device__ __forceinline__ void comp_put(Comp (&v)[N], int j, const Comp &c) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        v[i].s = (i == j) ? c.s : v[i].s;
        v[i].e = (i == j) ? c.e : v[i].e;
    }
}

// ------------------------------------------------------------------ attenuation
// One thread per ray, from the detector end: T the compensated suffix sum of m = W mu, att = exp(-L) of
// L_k = dx (m_k / 2 + T), the 4 samples of a group (k a multiple of 4) as one 16-byte store, padding rows 0.
// Bound by the stores (268M samples, 256 candidates at 128 pixels and 128 angles: 263 us, 4.1 TB/s; over 8
// lanes per ray, with its shuffles, 381 us).
// Row bands (!SINGLE): V is monotone along a ray, so the ray meets the bands in the order of its direction, and a
// workgroup takes rays of one direction (the first `up` of a candidate's chunks those along which V grows), dealt to
// the workgroups of that direction by waves: each band is staged once, and a ray keeps its sum and its open group in
// registers from band to band. Bound by its vector work; few rays by the stages' latency. 32 candidates at 256 pixels and
// 128 angles: 265 us; with both directions in a workgroup, so 2 bands - 1 stages of which a ray sits out all but `bands`,
// 277; storing m band by band and scanning it in a second pass 556. One candidate at 400 pixels and 20 angles: 283 us,
// 447 and 347.
template <bool SINGLE>
__device__ __forceinline__ void k_att_body(int bid, float *lds, DevGeom g, const Bands &bands, int rpt, int chunks, int up, int C,
                                             const float *__restrict__ mu, float *__restrict__ att, size_t img_cs,
                                             size_t att_cs, float *__restrict__ E, size_t e_cs) {
    int cand, chunk;
    ray_block(bid, chunks, C, cand, chunk);
    const int nrays = g.nah * g.nb;
    const int pitch = bands.pitch;
    const float nf = (float)g.n;
    const float *img = mu + cand * img_cs;
    float *out = att + cand * att_cs;

    if constexpr (SINGLE) {
        __syncthreads();  // the persistent executor's previous item
        stage_whole(img, g.n, bands.band(0, g.n), lds);
        __syncthreads();
        for (int j = 0; j < rpt; ++j) {
            const int ray = (chunk * rpt + j) * blockDim.x + threadIdx.x;
            if (ray >= nrays) break;
            const int a = ray / g.nb, b = ray - a * g.nb;
            const float2 cs = g.trig[a];
            float Ub, Vb;
            ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
            float *col = out + att_base(g, a, b);
            Comp T{0.f, 0.f};
            auto group = [&](auto whole, int kg) {
                float m[4], e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (decltype(whole)::value || 4 * kg + q < g.nt) {
                        float U, V;
                        sample_uv(Ub, Vb, tau_of(g, 4 * kg + q), cs.x, cs.y, U, V);
                        m[q] = bilinear_whole(lds, U, V, nf, pitch);
                    }
                }
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    e[q] = 0.f;
                    if (decltype(whole)::value || 4 * kg + q < g.nt) {
                        const float L = g.dx * (fmaf(0.5f, m[q], T.s) + T.e);
                        e[q] = fmaxf(expf(-L), kMinNormal);
                        comp_add(T, m[q]);
                    }
                }
                *reinterpret_cast<float4 *>(col + att_row(g, 4 * kg)) = make_float4(e[0], e[1], e[2], e[3]);
            };
            int kg = (g.nt - 1) >> 2;
            if ((g.nt & 3) != 0) group(std::false_type{}, kg--);
            for (; kg >= 0; --kg) group(std::true_type{}, kg);
            // opposed-ray pairing: exp(-T) of the whole ray, T = dx sum_k m_k
            if (E) E[cand * e_cs + ray] = expf(-g.dx * comp_value(T));
        }
    } else {
        // rays along which V grows with k (cos >= 0) take the last band first, the others the first
        const bool grows = chunk < up;
        const int mine = grows ? chunk : chunk - up, of = grows ? up : chunks - up;
        const AttAngles angles = att_angles(g.na, g.nah);
        const int rays = (grows ? angles.up : g.nah - angles.up) * g.nb;
        const int first = grows ? angles.first_up : angles.first_down;
        Comp T[kMaxRpt];
        float4 open[kMaxRpt];  // the open group: its samples so far
#pragma unroll
        for (int j = 0; j < kMaxRpt; ++j) {
            T[j] = Comp{0.f, 0.f};
            open[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int v = 0; v < bands.count; ++v) {
            const Band band = bands.band(grows ? bands.count - 1 - v : v, g.n);
            const BandTap bt = band_tap(band, nf, pitch);
            __syncthreads();
            stage_band<1>(img, g.n, band, lds);
            __syncthreads();
#pragma unroll 1
            for (int j = 0; j < rpt; ++j) {
                const int i = band_ray(mine, of, j);
                if (i >= rays) continue;
                const int p = i / g.nb, b = i - p * g.nb;
                const int a = first + p < g.nah ? first + p : first + p - g.nah, ray = a * g.nb + b;
                const float2 cs = g.trig[a];
                float Ub, Vb;
                ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
                int k0, k1;
                band_own_range(g, band, Vb, cs.x, k0, k1);
                float *col = out + att_base(g, a, b);
                Comp t = comp_pick(T, j);
                float4 o = open[0];
#pragma unroll
                for (int i = 1; i < kMaxRpt; ++i) {
                    o.x = (i == j) ? open[i].x : o.x;
                    o.y = (i == j) ? open[i].y : o.y;
                    o.z = (i == j) ? open[i].z : o.z;
                    o.w = (i == j) ? open[i].w : o.w;
                }
                for (int kg = (k0 <= k1) ? k1 & ~3 : -1; kg >= 0 && kg + 3 >= k0; kg -= 4) {
                    const unsigned bits = band_bits(kg, k0, k1);
                    float m[4], e[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float U, V, fu, fv;
                        sample_uv(Ub, Vb, tau_of(g, kg + q), cs.x, cs.y, U, V);
                        const int off = band_off(bt, U, V, nf, pitch, fu, fv);
                        m[q] = bit_keep(bits, q, lerp2(lds + off, pitch, fu, fv));
                    }
#pragma unroll
                    for (int q = 3; q >= 0; --q) {
                        const float L = g.dx * (fmaf(0.5f, m[q], t.s) + t.e);
                        e[q] = fmaxf(expf(-L), kMinNormal);
                        comp_add(t, m[q]);
                    }
                    o.x = (bits & 1u) ? e[0] : o.x;
                    o.y = (bits & 2u) ? e[1] : o.y;
                    o.z = (bits & 4u) ? e[2] : o.z;
                    o.w = (bits & 8u) ? e[3] : o.w;
                    if (kg >= k0) *reinterpret_cast<float4 *>(col + att_row(g, kg)) = o;
                }
                comp_put(T, j, t);
#pragma unroll
                for (int i = 0; i < kMaxRpt; ++i) {
                    open[i].x = (i == j) ? o.x : open[i].x;
                    open[i].y = (i == j) ? o.y : open[i].y;
                    open[i].z = (i == j) ? o.z : open[i].z;
                    open[i].w = (i == j) ? o.w : open[i].w;
                }
                if (E && v == bands.count - 1) E[cand * e_cs + ray] = expf(-g.dx * comp_value(t));
            }
        }
    }
}

#ifndef BOAC_BODIES_ONLY
template <bool SINGLE>
__global__ __launch_bounds__(1024) void k_att(DevGeom g, Bands bands, int rpt, int chunks, int up, int C,
                                             const float *__restrict__ mu, float *__restrict__ att, size_t img_cs,
                                             size_t att_cs, float *__restrict__ E, size_t e_cs) {
    extern __shared__ float lds[];
    k_att_body<SINGLE>(blockIdx.x, lds, g, bands, rpt, chunks, up, C, mu, att, img_cs, att_cs, E, e_cs);
}
#endif

// The same for few candidates: a ray's samples over kScanLanes lanes of one wave (single-stage images). The
// ray is walked from the detector end in rounds of kScanLanes 4-sample groups, lane j sampling the j-th group
// of the round; every lane then runs the round's compensated sum sample by sample, noting it where its own group
// begins, so every att has k_att's bits. The exponentials and stores are spread again; the 8 lanes of a ray and the
// 8 rays of a wave (consecutive bins) write whole 128-byte lines. passes: rays per lane group handled in turn, so
// that one image stage serves many rays.
constexpr int kScanLanes = 8;

#ifndef BOAC_BODIES_ONLY
// x of another lane by the data-parallel path; dpp_banks: in the 4-lane banks of BANKS only, elsewhere this lane's.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL, int BANKS>
__device__ __forceinline__ float dpp_banks(float x) {
    const int v = (int)__float_as_uint(x);
    return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, BANKS, false));
}
// sum + x of the ray's samples one by one, lane 0's x[3] to x[0] first, lane 7's last; returned: the sum before this
// lane's own. An addition reads the sample from its lane through the data-parallel path, which reaches the four lanes
// of a quad: the other quad's samples are brought to the same places first. (Each sample by a shuffle through the LDS
// unit, with its whole compensated step in every lane: one candidate at 128 pixels and 128 angles 12.8 us, 10.4 so;
// four 22.7, 19.1; eight at 64 and 64 9.2, 8.5.)
__device__ __forceinline__ float scan_run(float &sum, const float (&x)[4], int lane) {
    float half[2][4];  // the samples of lanes 0..3 and 4..7, by place in the quad
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        half[0][q] = dpp_banks<0x114, 0xa>(x[q]);  // lanes 4..7 of each 8: from 4 lanes below
        half[1][q] = dpp_banks<0x104, 0x5>(x[q]);  // lanes 0..3: from 4 lanes above
    }
    float own = sum;
    auto lane4 = [&](auto place, int h) {
        constexpr int p = decltype(place)::value;
        own = (lane == 4 * h + p) ? sum : own;
#pragma unroll
        for (int q = 3; q >= 0; --q) sum += dpp<p * 0x55>(half[h][q]);
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        lane4(std::integral_constant<int, 0>{}, h);
        lane4(std::integral_constant<int, 1>{}, h);
        lane4(std::integral_constant<int, 2>{}, h);
        lane4(std::integral_constant<int, 3>{}, h);
    }
    return own;
}

__global__ __launch_bounds__(256) void k_att_scan(DevGeom g, Band band, int passes, int chunks, int C,
                                                  const float *__restrict__ mu, float *__restrict__ att,
                                                  size_t img_cs, size_t att_cs, float *__restrict__ E,
                                                  size_t e_cs) {
    extern __shared__ float lds[];
    int cand, chunk;
    ray_block(blockIdx.x, chunks, C, cand, chunk);
    const int pitch = band.pitch;
    const float nf = (float)g.n;
    stage_whole<16>(mu + cand * img_cs, g.n, band, lds);
    __syncthreads();
    const int nrays = g.nah * g.nb;
    const int rpp = blockDim.x / kScanLanes;
    const int lane = threadIdx.x & (kScanLanes - 1);
    const int ng = (g.nt + 3) >> 2;
    const int rounds = (ng + kScanLanes - 1) / kScanLanes;
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(att + cand * att_cs, (unsigned)(4 * att_cs));
    for (int ps = 0; ps < passes; ++ps) {
        const int ray = (chunk * passes + ps) * rpp + (int)threadIdx.x / kScanLanes;
        const bool live = ray < nrays;
        const int a = live ? ray / g.nb : 0, b = live ? ray - a * g.nb : 0;
        const float2 cs = g.trig[a];
        float Ub, Vb;
        ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
        const unsigned roff = 4u * (unsigned)att_base(g, a, b);
        Comp T{0.f, 0.f};
        for (int r = 0; r < rounds; ++r) {
            const int grp = ng - 1 - (r * kScanLanes + lane);
            float m[4];
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                const int k = 4 * grp + q;
                float U, V;
                sample_uv(Ub, Vb, tau_of(g, k), cs.x, cs.y, U, V);
                const float w = bilinear_whole(lds, U, V, nf, pitch);
                m[q] = (live && grp >= 0 && k < g.nt) ? w : 0.f;  // no sample: adds nothing
            }
            // comp_add sample by sample in two runs: the sums s, whose roundings each lane finds for its own samples,
            // then the sums e of those
            float before[4], err[4], t = scan_run(T.s, m, lane);
#pragma unroll
            for (int q = 3; q >= 0; --q) {
                before[q] = t;
                two_sum(before[q], m[q], t, err[q]);
            }
            float own_e = scan_run(T.e, err, lane);
            if (live && grp >= 0) {
                float e[4];
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    const float L = g.dx * (fmaf(0.5f, m[q], before[q]) + own_e);
                    e[q] = (4 * grp + q < g.nt) ? fmaxf(expf(-L), kMinNormal) : 0.f;
                    own_e += err[q];
                }
                buffer_st4_stream(rs, roff + 4u * att_row(g, 4 * grp), 0u, make_float4(e[0], e[1], e[2], e[3]));
            }
        }
        if (E && live && lane == 0) E[cand * e_cs + ray] = expf(-g.dx * comp_value(T));
    }
}
#endif

// ------------------------------------------------------------------ forward projection
// The epilogue of one ray: y, or the MLEM ratio, or (returned) the NLL term; zero_proj is set where
// S > 0 meets y <= 0. S: the ray's measured count (unused in a plain projection).
template <int MODE>
__device__ __forceinline__ float fwd_meas(const FwdArgs &A, int ray) {
    return MODE == FWD_PROJ ? 0.f : A.meas[ray];
}
template <int MODE>
__device__ __forceinline__ float fwd_emit(const FwdArgs &A, size_t cand, int ray, float S, float y, bool &zero_proj) {
    const size_t si = cand * A.sino_cs + ray;
    if constexpr (MODE == FWD_PROJ) {
        A.y_out[si] = y;
        return 0.f;
    } else if constexpr (MODE == FWD_RATIO) {
        A.r_out[si] = (y > 0.f) ? S / y : 0.f;
        if (A.y_out) A.y_out[si] = y;
        return 0.f;
    } else {  // FWD_NLL
        if (A.y_out) A.y_out[si] = y;
        float term;
        if (S > 0.f) {
            if (y > 0.f) {
                // y - S ln y less its measurement-only part S - S ln S (summed with ln Gamma(S + 1) in the
                // likelihood constant): y - S - S ln(y / S), with y - S exact where y is within a factor
                // of 2 of S
                const float d = y - S;
                term = d - S * log1pf(d / S);
            } else if (y <= 0.f) {
                term = __builtin_inff();
                zero_proj = true;
            } else {
                term = y;  // NaN propagates (flagged as non-finite at the end)
            }
        } else {
            term = y;
        }
        return term;
    }
}

// 1 / att for the opposed ray's attenuation exp(-T) / att; att is clamped to the smallest normal
// float (exact for path lengths below ~87 optical depths).
__device__ __forceinline__ float inv_att(float at) { return rcp_clamped(at); }
__device__ __forceinline__ float opposed_att(float e_ray, float at) { return e_ray * inv_att(at); }

// One ray's samples in one row band: its projection (c) and, PAIRED, the opposed ray's (c2).
template <bool PAIRED>
__device__ __forceinline__ void fwd_band_ray(const DevGeom &g, const Band &band, const float *lds, const float *att,
                                             unsigned att_bytes, int a, int b, float2 cs, float Ub, float Vb, float e_ray,
                                             Comp &c, Comp &c2) {
    const int pitch = band.pitch;
    const float nf = (float)g.n;
    // The ray's samples in this band, KC at a time from the 4-aligned group holding the first, the next
    // chunk's loads (4 samples per 16-byte load) in flight meanwhile. The owned range is exact and the other
    // samples' values are masked, so a chunk has no branch and its LDS reads overlap (a test and a branch per
    // sample: each sample's LDS latency showed). Bound by the vector work, 28 operations a sample and a third
    // more where a wave's rays lie unevenly in a band. 32 candidates at 256 pixels and 128 angles: 251 us with
    // the branches, 213 without, 197 with the rays dealt out (band_ray).
    int k0, k1;
    band_own_range(g, band, Vb, cs.x, k0, k1);
    const BandTap bt = band_tap(band, nf, pitch);
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(att, att_bytes);
    const unsigned roff = 4u * (unsigned)att_base(g, a, b);
    if (k0 <= k1) {
        constexpr int KC = PAIRED ? 16 : 8, KG = KC / 4;
        // groups past the last are read again (in range; masked)
        float4 cur[KG], nxt[KG];
#pragma unroll
        for (int q = 0; q < KG; ++q)
            cur[q] = buffer_ld4(rs, roff + 4u * att_row(g, min((k0 & ~3) + 4 * q, k1 & ~3)), 0u);
        float tau = tau_of(g, k0 & ~3);
        for (int kc = k0 & ~3; kc <= k1; kc += KC) {
#pragma unroll
            for (int q = 0; q < KG; ++q)
                nxt[q] = buffer_ld4(rs, roff + 4u * att_row(g, min(kc + KC + 4 * q, k1 & ~3)), 0u);
            const unsigned bits = band_bits(kc, k0, k1);
            float part = 0.f, part2 = 0.f;
#pragma unroll
            for (int q = 0; q < KC; ++q) {
                float U, V, fu, fv;
                sample_uv(Ub, Vb, tau, cs.x, cs.y, U, V);
                const int off = band_off(bt, U, V, nf, pitch, fu, fv);
                const float at = f4at(cur[q >> 2], q & 3);
                const float w = bit_keep(bits, q, lerp2(lds + off, pitch, fu, fv));
                part = fmaf(at, w, part);
                if constexpr (PAIRED) part2 = fmaf(opposed_att(e_ray, at), w, part2);
                tau += 1.f;
            }
            kahan_add(c, part);
            if constexpr (PAIRED) kahan_add(c2, part2);
#pragma unroll
            for (int q = 0; q < KG; ++q) cur[q] = nxt[q];
        }
    }
}

// PAIRED (opposed-ray pairing): each thread's ray (a, b), a < na/2, also gives the
// projection of ray (a + na/2, nb-1-b) from the same samples and bilinear values.
template <int MODE, bool SINGLE, bool PAIRED>
__device__ __forceinline__ void k_fwd_body(int bid, float *lds, float *red, DevGeom g, const Bands &bands, int rpt, int chunks,
                                           int C, FwdArgs A) {
    int cand, chunk;
    ray_block(bid, chunks, C, cand, chunk);
    const int nrays = g.nah * g.nb;
    const int pitch = bands.pitch;
    const float nf = (float)g.n;
    const float *att = A.att + cand * A.att_cs;
    const float *img = A.img + cand * A.img_cs;
    Comp nll{0.f, 0.f};
    bool zero_proj = false;
    auto emit = [&](int ray, const Comp &c, const Comp &c2) {
        const float t0 = fwd_emit<MODE>(A, cand, ray, fwd_meas<MODE>(A, ray), g.dx * comp_value(c), zero_proj);
        if constexpr (MODE == FWD_NLL) comp_add(nll, t0);
        if constexpr (PAIRED) {
            const int a = ray / g.nb, b = ray - a * g.nb;
            const int opp = (a + g.nah) * g.nb + (g.nb - 1 - b);
            const float t1 = fwd_emit<MODE>(A, cand, opp, fwd_meas<MODE>(A, opp), g.dx * comp_value(c2), zero_proj);
            if constexpr (MODE == FWD_NLL) comp_add(nll, t1);
        }
    };

    if constexpr (!SINGLE) {
        Comp acc[kMaxRpt], acc2[PAIRED ? kMaxRpt : 1];
#pragma unroll
        for (int j = 0; j < kMaxRpt; ++j) acc[j] = Comp{0.f, 0.f};
#pragma unroll
        for (int j = 0; j < (PAIRED ? kMaxRpt : 1); ++j) acc2[j] = Comp{0.f, 0.f};
        for (int bi = 0; bi < bands.count; ++bi) {
            const Band band = bands.band(bi, g.n);
            __syncthreads();
            if (A.img_comps == 1)
                stage_band<1>(img, g.n, band, lds);
            else
                stage_band_strided(img, g.n, A.img_comps, band, lds);  // component 0 of an interleaved pair
            __syncthreads();
            // one copy of the loop body: unrolled over the rays it would outgrow the registers
#pragma unroll 1
            for (int j = 0; j < rpt; ++j) {
                const int ray = band_ray(chunk, chunks, j);
                if (ray >= nrays) continue;
                const int a = ray / g.nb, b = ray - a * g.nb;
                const float2 cs = g.trig[a];
                float Ub, Vb;
                ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
                Comp c = comp_pick(acc, j), c2{0.f, 0.f};
                if constexpr (PAIRED) c2 = comp_pick(acc2, j);
                fwd_band_ray<PAIRED>(g, band, lds, att, (unsigned)(4 * A.att_cs), a, b, cs, Ub, Vb,
                                     PAIRED ? A.E[cand * A.e_cs + ray] : 0.f, c, c2);
                comp_put(acc, j, c);
                if constexpr (PAIRED) comp_put(acc2, j, c2);
            }
        }
#pragma unroll
        for (int j = 0; j < kMaxRpt; ++j) {
            if (j >= rpt) break;
            const int ray = band_ray(chunk, chunks, j);
            if (ray < nrays) emit(ray, acc[j], acc2[PAIRED ? j : 0]);
        }
    } else {
        __syncthreads();
        if (A.img_comps == 1)
            stage_band<1>(img, g.n, bands.band(0, g.n), lds);
        else
            stage_band_strided(img, g.n, A.img_comps, bands.band(0, g.n), lds);  // component 0 of an interleaved pair
        __syncthreads();
        // att is streamed 16 samples ahead of use: the loads of chunk k0 + 16 are in flight while chunk k0 is
        // computed. The loads go through a buffer resource: a per-lane ray offset plus a uniform offset of the
        // sample row; each 16-byte load brings 4 consecutive samples of the ray (one group of the layout).
        // Each chunk is summed with FMAs and added to the compensated total. A whole chunk has no branch, so
        // its samples' LDS reads overlap; the samples past the last whole chunk are tested one by one. (A test
        // per sample showed every LDS read's latency: projection of candidate pairs, 64 at 128 pixels and 72
        // angles 42.2 us, 39.5 without; reverse sweep of 64 at 128 angles 136, 128 without.)
        const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(att, (unsigned)(4 * A.att_cs));
#pragma unroll 1
        for (int j = 0; j < rpt; ++j) {
            const int ray = (chunk * rpt + j) * blockDim.x + threadIdx.x;
            if (ray >= nrays) break;
            const int a = ray / g.nb, b = ray - a * g.nb;
            const float2 cs = g.trig[a];
            float Ub, Vb;
            ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
            const unsigned roff = 4u * (unsigned)att_base(g, a, b);
            const float e_ray = PAIRED ? A.E[cand * A.e_cs + ray] : 0.f;
            Comp c{0.f, 0.f}, c2{0.f, 0.f};
            float4 cur[kRayGroups], nxt[kRayGroups];
            float tau = -g.cT;
            auto load = [&](int k0, float4 *v) {  // groups past the ray's last: that one again (not used)
#pragma unroll
                for (int q = 0; q < kRayGroups; ++q) v[q] = buffer_ld4_stream(rs, roff, 4u * att_row(g, ray_group(g, k0, q)));
            };
            auto sum = [&](auto whole, int k0) {
                float part = 0.f, part2 = 0.f;
#pragma unroll
                for (int q = 0; q < kRayChunk; ++q) {
                    if (decltype(whole)::value || k0 + q < g.nt) {
                        float U, V;
                        sample_uv(Ub, Vb, tau, cs.x, cs.y, U, V);
                        const float at = f4at(cur[q >> 2], q & 3);
                        const float w = bilinear_whole(lds, U, V, nf, pitch);
                        part = fmaf(at, w, part);
                        if constexpr (PAIRED) part2 = fmaf(opposed_att(e_ray, at), w, part2);
                    }
                    tau += 1.f;
                }
                kahan_add(c, part);
                if constexpr (PAIRED) kahan_add(c2, part2);
            };
            load(0, cur);
            int k0 = 0;
            for (; k0 + kRayChunk <= g.nt; k0 += kRayChunk) {
                if (k0 + kRayChunk < g.nt) load(k0 + kRayChunk, nxt);
                sum(std::true_type{}, k0);
#pragma unroll
                for (int q = 0; q < kRayGroups; ++q) cur[q] = nxt[q];
            }
            if (k0 < g.nt) sum(std::false_type{}, k0);
            emit(ray, c, c2);
        }
    }
    if constexpr (MODE == FWD_NLL) {
        if (zero_proj && A.status) atomicOr(A.status + cand, 1u);
        const Comp r = block_reduce(nll, red);
        if (threadIdx.x == 0) A.partial[(size_t)cand * chunks + chunk] = make_float2(r.s, r.e);
    }
}

#ifndef BOAC_BODIES_ONLY
template <int MODE, bool SINGLE, bool PAIRED>
__global__ __launch_bounds__(1024) void k_fwd(DevGeom g, Bands bands, int rpt, int chunks, int C, FwdArgs A) {
    extern __shared__ float lds[];
    __shared__ float red[32];  // two floats per wave, up to 16 waves
    k_fwd_body<MODE, SINGLE, PAIRED>(blockIdx.x, lds, red, g, bands, rpt, chunks, C, A);
}
#endif

// Forward projection of two candidates per workgroup, both images staged at once (interleaved as
// float2): each sample's position, clamp, tap index and bilinear fractions are computed once and
// serve both candidates (one pair lerp, two FMAs), about half the vector work per candidate-sample of
// k_fwd. Single-stage images only (the pair stage is twice the size). An odd batch's last pair
// repeats its candidate and writes it once. PAIRED: opposed-ray pairing as in k_fwd.
template <int MODE, bool PAIRED>
__device__ __forceinline__ void k_fwd_pair_body(int bid, float *lds, float *red, DevGeom g, const Bands &bands, int rpt, int chunks, int C, FwdArgs A) {
    const int npairs = (C + 1) >> 1;
    int pr, chunk;
    ray_block(bid, chunks, npairs, pr, chunk);
    const int c0 = 2 * pr;
    const bool two = (c0 + 1 < C);
    const int c1 = two ? c0 + 1 : c0;
    const int nrays = g.nah * g.nb;
    const int pitch = bands.pitch;
    const float nf = (float)g.n;
    stage_band_pair(A.img + c0 * A.img_cs, A.img + c1 * A.img_cs, g.n, bands.band(0, g.n), lds);
    __syncthreads();
    const float2 *lds2 = reinterpret_cast<const float2 *>(lds);
    const __amdgpu_buffer_rsrc_t r0 = buffer_rsrc(A.att + c0 * A.att_cs, (unsigned)(4 * A.att_cs));
    const __amdgpu_buffer_rsrc_t r1 = buffer_rsrc(A.att + c1 * A.att_cs, (unsigned)(4 * A.att_cs));

    Comp nll[2] = {{0.f, 0.f}, {0.f, 0.f}};
    bool zero_proj[2] = {false, false};
#pragma unroll 1
    for (int j = 0; j < rpt; ++j) {
        const int ray = (chunk * rpt + j) * blockDim.x + threadIdx.x;
        if (ray >= nrays) break;
        const int a = ray / g.nb, b = ray - a * g.nb;
        const float2 cs = g.trig[a];
        float Ub, Vb;
        ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
        const unsigned roff = 4u * (unsigned)att_base(g, a, b);
        const float e0 = PAIRED ? A.E[c0 * A.e_cs + ray] : 0.f;
        const float e1 = PAIRED ? A.E[c1 * A.e_cs + ray] : 0.f;
        // 8 samples ahead (16 would not leave the registers for overlapping LDS reads): the first half of a
        // chunk in x, the second in y
        constexpr int KH = kRayChunk / 2, HG = KH / 4;
        float4 x0[HG], x1[HG], y0[HG], y1[HG];
        Comp s0{0.f, 0.f}, s1{0.f, 0.f}, t0{0.f, 0.f}, t1{0.f, 0.f};
        float tau = -g.cT;
        auto load = [&](int k0, float4 *v0, float4 *v1) {
#pragma unroll
            for (int q = 0; q < HG; ++q) {
                const unsigned o = 4u * att_row(g, ray_group(g, k0, q));
                v0[q] = buffer_ld4_stream(r0, roff, o);
                v1[q] = buffer_ld4_stream(r1, roff, o);
            }
        };
        float p0, p1, o0, o1;
        auto sum = [&](auto whole, int k0, const float4 *v0, const float4 *v1) {
#pragma unroll
            for (int q = 0; q < KH; ++q) {
                if (decltype(whole)::value || k0 + q < g.nt) {
                    float U, V;
                    sample_uv(Ub, Vb, tau, cs.x, cs.y, U, V);
                    const float Uc = __builtin_amdgcn_fmed3f(U, -1.f, nf);
                    const float Vc = __builtin_amdgcn_fmed3f(V, -1.f, nf);
                    const int idx = (int)fmaf(floorf(Vc), (float)pitch, floorf(Uc));
                    const float2 w = lerp2x2(lds2 + idx + (pitch + 1), pitch, __builtin_amdgcn_fractf(Uc),
                                             __builtin_amdgcn_fractf(Vc));
                    const float a0 = f4at(v0[q >> 2], q & 3), a1 = f4at(v1[q >> 2], q & 3);
                    p0 = fmaf(a0, w.x, p0);
                    p1 = fmaf(a1, w.y, p1);
                    if constexpr (PAIRED) {
                        o0 = fmaf(opposed_att(e0, a0), w.x, o0);
                        o1 = fmaf(opposed_att(e1, a1), w.y, o1);
                    }
                }
                tau += 1.f;
                if ((q & 3) == 3) {
                    // the sums so far are due here: otherwise every sample's LDS reads of the half are issued
                    // first, and what they return outgrows the registers
                    if constexpr (PAIRED) asm volatile("" : "+v"(o0), "+v"(o1));
                    asm volatile("" : "+v"(p0), "+v"(p1)::"memory");
                }
            }
        };
        auto chunk_end = [&]() {
            kahan_add(s0, p0);
            kahan_add(s1, p1);
            if constexpr (PAIRED) {
                kahan_add(t0, o0);
                kahan_add(t1, o1);
            }
        };
        load(0, x0, x1);
        int k0 = 0;
        for (; k0 + kRayChunk <= g.nt; k0 += kRayChunk) {
            p0 = p1 = o0 = o1 = 0.f;
            load(k0 + KH, y0, y1);
            sum(std::true_type{}, k0, x0, x1);
            if (k0 + kRayChunk < g.nt) load(k0 + kRayChunk, x0, x1);
            sum(std::true_type{}, k0 + KH, y0, y1);
            chunk_end();
        }
        if (k0 < g.nt) {
            p0 = p1 = o0 = o1 = 0.f;
            load(k0 + KH, y0, y1);
            sum(std::false_type{}, k0, x0, x1);
            sum(std::false_type{}, k0 + KH, y0, y1);
            chunk_end();
        }
        // epilogues, candidate by candidate
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 1 && !two) break;
            const int cand = h ? c1 : c0;
            const float z0 = fwd_emit<MODE>(A, cand, ray, fwd_meas<MODE>(A, ray), g.dx * comp_value(h ? s1 : s0), zero_proj[h]);
            if constexpr (MODE == FWD_NLL) comp_add(nll[h], z0);
            if constexpr (PAIRED) {
                const int opp = (a + g.nah) * g.nb + (g.nb - 1 - b);
                const float z1 =
                    fwd_emit<MODE>(A, cand, opp, fwd_meas<MODE>(A, opp), g.dx * comp_value(h ? t1 : t0), zero_proj[h]);
                if constexpr (MODE == FWD_NLL) comp_add(nll[h], z1);
            }
        }
    }
    if constexpr (MODE == FWD_NLL) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int cand = h ? c1 : c0;
            const bool live = (h == 0) || two;
            if (zero_proj[h] && A.status) atomicOr(A.status + cand, 1u);
            const Comp r = block_reduce(nll[h], red);
            if (threadIdx.x == 0 && live) A.partial[(size_t)cand * chunks + chunk] = make_float2(r.s, r.e);
        }
    }
}

#ifndef BOAC_BODIES_ONLY
template <int MODE, bool PAIRED>
__global__ __launch_bounds__(1024) void k_fwd_pair(DevGeom g, Bands bands, int rpt, int chunks, int C, FwdArgs A) {
    extern __shared__ float lds[];
    __shared__ float red[32];  // two floats per wave, up to 16 waves
    k_fwd_pair_body<MODE, PAIRED>(blockIdx.x, lds, red, g, bands, rpt, chunks, C, A);
}
#endif

// ------------------------------------------------------------------ fused reverse sweep
// One ray's samples in one row band of a reverse step: r_bar of the ray (c) and, PAIRED, of the opposed ray
// (c2) and the ray's E_bar part (eb); att_bar is read and written. rr, yp (rr2, yp2 opposed): dx r and dx ybar.
template <bool PAIRED>
__device__ __forceinline__ void sweep_band_ray(const DevGeom &g, const Band &band, const float2 *lds2,
                                               __amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb, int accumulate, int a, int b, float2 cs,
                                               float Ub, float Vb, float e_ray, float rr, float yp, float rr2, float yp2,
                                               Comp &c, Comp &c2, Comp &eb) {
    const int pitch = band.pitch;
    const float nf = (float)g.n;
    // The ray's samples in this band as in the projection: exact range, masked values, 8 at a time (the most
    // whose att and att_bar, this chunk's and the next one's, fit the registers). The ray is this thread's alone
    // and its bands run in order, so a group's samples owned by another band are written back as loaded.
    // Bound by the vector work, as the projection; 32 candidates at 256 pixels and 128 angles: 601 us.
    int k0, k1;
    band_own_range(g, band, Vb, cs.x, k0, k1);
    const BandTap btap = band_tap(band, nf, pitch);
    const unsigned roff = 4u * (unsigned)att_base(g, a, b);
    if (k0 <= k1) {
        constexpr int KC = 8, KG = KC / 4;
        const int kl = k1 & ~3;  // the last group
        float4 av[KG], an[KG], bv[KG], bn[KG];
#pragma unroll
        for (int q = 0; q < KG; ++q) {
            const unsigned o = roff + 4u * att_row(g, min((k0 & ~3) + 4 * q, kl));
            av[q] = buffer_ld4(ra, o, 0u);
            bv[q] = buffer_ld4(rb, o, 0u);
        }
        float tau = tau_of(g, k0 & ~3);
        for (int kc = k0 & ~3; kc <= k1; kc += KC) {
            // (the last chunk reads its last group again before it is stored: not used)
#pragma unroll
            for (int q = 0; q < KG; ++q) {
                const unsigned o = roff + 4u * att_row(g, min(kc + KC + 4 * q, kl));
                an[q] = buffer_ld4(ra, o, 0u);
                bn[q] = buffer_ld4(rb, o, 0u);
            }
            const unsigned bits = band_bits(kc, k0, k1);
            const unsigned drop = accumulate ? 0u : bits;  // first write: att_bar's old value goes
            float part = 0.f, part2 = 0.f, epart = 0.f;
            float ov[4];
#pragma unroll
            for (int q = 0; q < KC; ++q) {
                float U, V, fu, fv;
                sample_uv(Ub, Vb, tau, cs.x, cs.y, U, V);
                const int off = band_off(btap, U, V, nf, pitch, fu, fv);
                float2 w = lerp2x2(lds2 + off, pitch, fu, fv);
                w.x = bit_keep(bits, q, w.x);
                w.y = bit_keep(bits, q, w.y);
                const float a0 = f4at(av[q >> 2], q & 3);
                part = fmaf(a0, w.x, part);
                float d = fmaf(rr, w.x, yp * w.y);
                if constexpr (PAIRED) {
                    const float ri = inv_att(a0);
                    const float ao = e_ray * ri;
                    const float cv2 = fmaf(rr2, w.x, yp2 * w.y);
                    part2 = fmaf(ao, w.x, part2);
                    epart = fmaf(cv2, ri, epart);
                    d = fmaf(-ao * ri, cv2, d);
                }
                ov[q & 3] = bit_keep(~drop, q, f4at(bv[q >> 2], q & 3)) + bit_keep(bits, q, d);
                tau += 1.f;
                if ((q & 3) == 3 && kc + q - 3 <= k1)
                    buffer_st4(rb, roff + 4u * att_row(g, kc + q - 3), 0u,
                               make_float4(ov[0], ov[1], ov[2], ov[3]));
            }
            kahan_add(c, part);
            if constexpr (PAIRED) {
                kahan_add(c2, part2);
                kahan_add(eb, epart);
            }
#pragma unroll
            for (int q = 0; q < KG; ++q) {
                av[q] = an[q];
                bv[q] = bn[q];
            }
        }
    }
}

// One reverse MLEM step n, per ray i (pair image = (bbar^n, F^{n+1}) staged in LDS):
//   rbar_i   = dx sum_k att_ik (W bbar^n)_ik                          (adjoint of b^n = A^T r^n)
//   attbar_ik (+)= dx [ r^n_i (W bbar^n)_ik + ybar^{n+1}_i (W F^{n+1})_ik ]
//   ybar^n_i = -rbar_i r^n_i / y^n_i   (0 where y^n_i <= 0)               (adjoint of r = S / y)
// The ybar^{n+1} term is the y^{n+1} = A F^{n+1} adjoint left pending by the previous step (or the
// objective's adjoint for the first step), so each step sweeps the rays once.
// PAIRED (opposed-ray pairing): the held ray i also carries the opposed ray i', whose
// attenuation at the shared sample is att' = exp(-T) / att; its r_bar and ybar are formed the same
// way, and its attenuation adjoint c' = dx [ r^n_i' W bbar + ybar^{n+1}_i' W F^{n+1} ] reaches the
// held tensors through att' = E / att: att_bar += -att' c' / att, E_bar += c' / att.
template <bool SINGLE, bool PAIRED>
__device__ __forceinline__ void k_adj_sweep_body(int bid, float *lds, DevGeom g, const Bands &bands, int rpt, int chunks, int C, SweepArgs A) {
    int cand, chunk;
    ray_block(bid, chunks, C, cand, chunk);
    const int nrays = g.nah * g.nb;
    const int pitch = bands.pitch;
    const float nf = (float)g.n;
    const float *att = A.att + cand * A.att_cs;
    float *ab = A.attbar + cand * A.att_cs;
    const float *img = A.pair + cand * A.img_cs;
    const float2 *lds2 = reinterpret_cast<const float2 *>(lds);

    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(att, (unsigned)(4 * A.att_cs));
    const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(ab, (unsigned)(4 * A.att_cs));
    auto emit = [&](int ray, const Comp &c, const Comp &c2, const Comp &eb) {
        const size_t si = cand * A.sino_cs + ray;
        const float rbar = g.dx * comp_value(c);
        const float yn = A.y[si];
        A.ybar_out[si] = (yn > 0.f) ? -(rbar * A.r[si]) / yn : 0.f;
        if constexpr (PAIRED) {
            const int a = ray / g.nb, b = ray - a * g.nb;
            const size_t si2 = cand * A.sino_cs + (size_t)((a + g.nah) * g.nb + (g.nb - 1 - b));
            const float rbar2 = g.dx * comp_value(c2);
            const float yn2 = A.y[si2];
            A.ybar_out[si2] = (yn2 > 0.f) ? -(rbar2 * A.r[si2]) / yn2 : 0.f;
            float *eo = A.Ebar + cand * A.e_cs + ray;
            *eo = (A.accumulate ? *eo : 0.f) + comp_value(eb);
        }
    };
    if constexpr (!SINGLE) {
        // R rays' sums in registers at a time, the image staged again for the next ones
        constexpr int R = kSweepBandRpt;
        for (int j0 = 0; j0 < rpt; j0 += R) {
            Comp acc[R], acc2[R], ebj[R];  // PAIRED: r_bar of the opposed ray, its E_bar part
#pragma unroll
            for (int j = 0; j < R; ++j) acc[j] = acc2[j] = ebj[j] = Comp{0.f, 0.f};
            for (int bi = 0; bi < bands.count; ++bi) {
                const Band band = bands.band(bi, g.n);
                __syncthreads();
                stage_band<2>(img, g.n, band, lds);
                __syncthreads();
#pragma unroll 1
                for (int j = 0; j < min(rpt - j0, R); ++j) {
                    const int ray = band_ray(chunk, chunks, j0 + j);
                    if (ray >= nrays) continue;
                    const int a = ray / g.nb, b = ray - a * g.nb;
                    const float2 cs = g.trig[a];
                    float Ub, Vb;
                    ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
                    const size_t si = cand * A.sino_cs + ray;
                    const size_t si2 = cand * A.sino_cs + (size_t)((a + g.nah) * g.nb + (g.nb - 1 - b));
                    Comp c = comp_pick(acc, j), c2{0.f, 0.f}, eb{0.f, 0.f};
                    if constexpr (PAIRED) {
                        c2 = comp_pick(acc2, j);
                        eb = comp_pick(ebj, j);
                    }
                    sweep_band_ray<PAIRED>(g, band, lds2, ra, rb, A.accumulate, a, b, cs, Ub, Vb,
                                           PAIRED ? A.E[cand * A.e_cs + ray] : 0.f, g.dx * A.r[si], g.dx * A.ybar_in[si],
                                           PAIRED ? g.dx * A.r[si2] : 0.f, PAIRED ? g.dx * A.ybar_in[si2] : 0.f, c, c2,
                                           eb);
                    comp_put(acc, j, c);
                    if constexpr (PAIRED) {
                        comp_put(acc2, j, c2);
                        comp_put(ebj, j, eb);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (j0 + j >= rpt) break;
                const int ray = band_ray(chunk, chunks, j0 + j);
                if (ray < nrays) emit(ray, acc[j], acc2[j], ebj[j]);
            }
        }
    } else {
        __syncthreads();
        stage_band<2>(img, g.n, bands.band(0, g.n), lds);
        __syncthreads();
        // as in the forward projection: att and att_bar streamed 8 samples ahead through buffer resources,
        // chunked compensated sums, no branch in a whole chunk; padding rows of att_bar get 0
#pragma unroll 1
        for (int j = 0; j < rpt; ++j) {
            const int ray = (chunk * rpt + j) * blockDim.x + threadIdx.x;
            if (ray >= nrays) break;
            const int a = ray / g.nb, b = ray - a * g.nb;
            const float2 cs = g.trig[a];
            float Ub, Vb;
            ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
            const size_t si = cand * A.sino_cs + ray;
            const size_t si2 = cand * A.sino_cs + (size_t)((a + g.nah) * g.nb + (g.nb - 1 - b));
            const float rr = g.dx * A.r[si], yp = g.dx * A.ybar_in[si];
            const float e_ray = PAIRED ? A.E[cand * A.e_cs + ray] : 0.f;
            const float rr2 = PAIRED ? g.dx * A.r[si2] : 0.f;
            const float yp2 = PAIRED ? g.dx * A.ybar_in[si2] : 0.f;
            const unsigned roff = 4u * (unsigned)att_base(g, a, b);
            const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
            constexpr int KH = kRayChunk / 2, HG = KH / 4;
            float4 xa[HG], xb[HG], ya[HG], yb[HG];  // the halves of a chunk
            Comp c{0.f, 0.f}, c2{0.f, 0.f}, eb{0.f, 0.f};
            float tau = -g.cT;
            auto load = [&](int k0, float4 *va, float4 *vb) {
#pragma unroll
                for (int q = 0; q < HG; ++q) va[q] = buffer_ld4_stream(ra, roff, 4u * att_row(g, ray_group(g, k0, q)));
                if (A.accumulate) {
#pragma unroll
                    for (int q = 0; q < HG; ++q)
                        vb[q] = buffer_ld4_stream(rb, roff, 4u * att_row(g, ray_group(g, k0, q)));
                } else {
#pragma unroll
                    for (int q = 0; q < HG; ++q) vb[q] = z4;
                }
            };
            float part, part2, epart;
            auto step = [&](auto whole, int k0, const float4 *at, const float4 *bt) {
                constexpr bool kWhole = decltype(whole)::value;
                float ov[4];
#pragma unroll
                for (int q = 0; q < KH; ++q) {
                    const int k = k0 + q;
                    ov[q & 3] = 0.f;
                    if (kWhole || k < g.nt) {
                        float U, V;
                        sample_uv(Ub, Vb, tau, cs.x, cs.y, U, V);
                        const float Uc = __builtin_amdgcn_fmed3f(U, -1.f, nf);
                        const float Vc = __builtin_amdgcn_fmed3f(V, -1.f, nf);
                        const int idx = (int)fmaf(floorf(Vc), (float)pitch, floorf(Uc));
                        const float2 w = lerp2x2(lds2 + idx + (pitch + 1), pitch, __builtin_amdgcn_fractf(Uc),
                                                 __builtin_amdgcn_fractf(Vc));
                        const float a0 = f4at(at[q >> 2], q & 3);
                        part = fmaf(a0, w.x, part);
                        const float cv = fmaf(rr, w.x, yp * w.y);
                        if constexpr (PAIRED) {
                            const float ri = inv_att(a0);
                            const float ao = e_ray * ri;
                            const float cv2 = fmaf(rr2, w.x, yp2 * w.y);
                            part2 = fmaf(ao, w.x, part2);
                            epart = fmaf(cv2, ri, epart);
                            ov[q & 3] = f4at(bt[q >> 2], q & 3) + fmaf(-ao * ri, cv2, cv);
                        } else {
                            ov[q & 3] = f4at(bt[q >> 2], q & 3) + cv;
                        }
                    }
                    tau += 1.f;
                    if ((q & 3) == 3 && (kWhole || k - 3 < g.nt))
                        buffer_st4_stream(rb, roff, 4u * att_row(g, k - 3), make_float4(ov[0], ov[1], ov[2], ov[3]));
                }
            };
            auto chunk_end = [&]() {
                kahan_add(c, part);
                if constexpr (PAIRED) {
                    kahan_add(c2, part2);
                    kahan_add(eb, epart);
                }
            };
            load(0, xa, xb);
            int k0 = 0;
            for (; k0 + kRayChunk <= g.nt; k0 += kRayChunk) {
                part = part2 = epart = 0.f;
                load(k0 + KH, ya, yb);
                step(std::true_type{}, k0, xa, xb);
                if (k0 + kRayChunk < g.nt) load(k0 + kRayChunk, xa, xb);
                step(std::true_type{}, k0 + KH, ya, yb);
                chunk_end();
            }
            if (k0 < g.nt) {
                part = part2 = epart = 0.f;
                load(k0 + KH, ya, yb);
                step(std::false_type{}, k0, xa, xb);
                step(std::false_type{}, k0 + KH, ya, yb);
                chunk_end();
            }
            emit(ray, c, c2, eb);
        }
    }
}

#ifndef BOAC_BODIES_ONLY
template <bool SINGLE, bool PAIRED>
__global__ __launch_bounds__(1024) void k_adj_sweep(DevGeom g, Bands bands, int rpt, int chunks, int C, SweepArgs A) {
    extern __shared__ float lds[];
    k_adj_sweep_body<SINGLE, PAIRED>(blockIdx.x, lds, g, bands, rpt, chunks, C, A);
}
#endif

// ------------------------------------------------------------------ tail of the attenuation adjoint
// att_bar (+)= dx (W G1 + rho_i W G2) with the pair image (G1, G2) = (s_bar, F^0) and rho = ybar^0
// (the sensitivity adjoint and the last pending projection adjoint); then
// L_bar = -att * att_bar and m_bar_k = dx (L_bar_k / 2 + sum_{k'<k} L_bar_k') (the scan's transpose),
// written in place of att_bar.
// PAIRED (opposed-ray pairing): the opposed ray's part c' = dx (W G1 + rho_i' W G2)
// reaches att_bar and E_bar as in the sweep; at the ray's end Tbar = -E E_bar (E = exp(-T)), and
// since T = dx sum_k m_k every sample's m_bar gains dx Tbar, written per ray in place of E_bar (the
// field gather adds it).
template <bool SINGLE, bool PAIRED>
__device__ __forceinline__ void k_tail_body(int bid, float *lds, DevGeom g, const Bands &bands, int rpt, int chunks, int C, TailArgs A) {
    int cand, chunk;
    ray_block(bid, chunks, C, cand, chunk);
    const int nrays = g.nah * g.nb;
    const int pitch = bands.pitch;
    const float nf = (float)g.n;
    const float *att = A.att + cand * A.att_cs;
    float *ab = A.attbar + cand * A.att_cs;
    const float *img = A.pair + cand * A.img_cs;
    const float2 *lds2 = reinterpret_cast<const float2 *>(lds);
    Comp ebj[kMaxRpt];  // PAIRED, row bands: the opposed ray's E_bar part, summed over the bands
#pragma unroll
    for (int j = 0; j < kMaxRpt; ++j) ebj[j] = Comp{0.f, 0.f};

    for (int bi = 0; bi < bands.count; ++bi) {
        const Band band = bands.band(bi, g.n);
        __syncthreads();
        stage_band<2>(img, g.n, band, lds);
        __syncthreads();
#pragma unroll 1
        for (int j = 0; j < rpt; ++j) {
            const int ray = SINGLE ? (chunk * rpt + j) * (int)blockDim.x + (int)threadIdx.x : band_ray(chunk, chunks, j);
            if (ray >= nrays) continue;
            const int a = ray / g.nb, b = ray - a * g.nb;
            const float2 cs = g.trig[a];
            float Ub, Vb;
            ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
            const float rho = A.rho[cand * A.sino_cs + ray];
            const size_t off = att_base(g, a, b);
            if constexpr (SINGLE) {
                // samples move in groups of 4 (one 16-byte load or store); padding rows get 0
                // 8 ahead, and no test per sample in a whole chunk, as in the sweep
                const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(att, (unsigned)(4 * A.att_cs));
                const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(ab, (unsigned)(4 * A.att_cs));
                const unsigned roff = 4u * (unsigned)off;
                const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
                constexpr int KH = kRayChunk / 2, HG = KH / 4;
                float4 xa[HG], xb[HG], ya[HG], yb[HG];
                Comp P{0.f, 0.f};
                const float e_ray = PAIRED ? A.E[cand * A.e_cs + ray] : 0.f;
                const float rho2 =
                    PAIRED ? A.rho[cand * A.sino_cs + (size_t)((a + g.nah) * g.nb + (g.nb - 1 - b))] : 0.f;
                Comp eb{0.f, 0.f};
                float tau = -g.cT, epart;
                auto load = [&](int k0, float4 *va, float4 *vb) {
#pragma unroll
                    for (int q = 0; q < HG; ++q) {
                        const unsigned o = 4u * att_row(g, ray_group(g, k0, q));
                        va[q] = buffer_ld4_stream(ra, roff, o);
                        vb[q] = A.accumulate ? buffer_ld4_stream(rb, roff, o) : z4;
                    }
                };
                auto step = [&](auto whole, int k0, const float4 *at, const float4 *bt) {
                    constexpr bool kWhole = decltype(whole)::value;
                    float ov[4];
#pragma unroll
                    for (int q = 0; q < KH; ++q) {
                        const int k = k0 + q;
                        ov[q & 3] = 0.f;
                        if (kWhole || k < g.nt) {
                            float U, V;
                            sample_uv(Ub, Vb, tau, cs.x, cs.y, U, V);
                            const float Uc = __builtin_amdgcn_fmed3f(U, -1.f, nf);
                            const float Vc = __builtin_amdgcn_fmed3f(V, -1.f, nf);
                            const int idx = (int)fmaf(floorf(Vc), (float)pitch, floorf(Uc));
                            const float2 w = lerp2x2(lds2 + idx + (pitch + 1), pitch, __builtin_amdgcn_fractf(Uc),
                                                     __builtin_amdgcn_fractf(Vc));
                            const float a0 = f4at(at[q >> 2], q & 3);
                            float abar;
                            if constexpr (PAIRED) {
                                const float ri = inv_att(a0);
                                const float ao = e_ray * ri;
                                const float cv2 = g.dx * fmaf(rho2, w.y, w.x);
                                epart = fmaf(cv2, ri, epart);
                                abar = f4at(bt[q >> 2], q & 3) + fmaf(-ao * ri, cv2, g.dx * fmaf(rho, w.y, w.x));
                            } else {
                                abar = f4at(bt[q >> 2], q & 3) + g.dx * fmaf(rho, w.y, w.x);
                            }
                            const float Lbar = -a0 * abar;
                            ov[q & 3] = g.dx * (fmaf(0.5f, Lbar, P.s) + P.e);
                            comp_add(P, Lbar);
                        }
                        tau += 1.f;
                        if ((q & 3) == 3 && (kWhole || k - 3 < g.nt))
                            buffer_st4_stream(rb, roff, 4u * att_row(g, k - 3), make_float4(ov[0], ov[1], ov[2], ov[3]));
                    }
                };
                load(0, xa, xb);
                int k0 = 0;
                for (; k0 + kRayChunk <= g.nt; k0 += kRayChunk) {
                    epart = 0.f;
                    load(k0 + KH, ya, yb);
                    step(std::true_type{}, k0, xa, xb);
                    if (k0 + kRayChunk < g.nt) load(k0 + kRayChunk, xa, xb);
                    step(std::true_type{}, k0 + KH, ya, yb);
                    if constexpr (PAIRED) kahan_add(eb, epart);
                }
                if (k0 < g.nt) {
                    epart = 0.f;
                    load(k0 + KH, ya, yb);
                    step(std::false_type{}, k0, xa, xb);
                    step(std::false_type{}, k0 + KH, ya, yb);
                    if constexpr (PAIRED) kahan_add(eb, epart);
                }
                if constexpr (PAIRED) {
                    float *eo = A.Ebar + cand * A.e_cs + ray;
                    const float etot = (A.accumulate ? *eo : 0.f) + comp_value(eb);
                    *eo = g.dx * (-e_ray * etot);
                }
            } else {
                // pass 1 of 2 (band by band): att_bar (+)= dx (W G1 + rho W G2), 16 samples at a time
                // (from the 4-aligned group holding the first sample, 16-byte loads and stores; samples of
                // another band are written back as loaded, as in the sweep)
                int k0, k1;
                band_k_range(g, band, Vb, cs.x, k0, k1);
                const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(att, (unsigned)(4 * A.att_cs));
                const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(ab, (unsigned)(4 * A.att_cs));
                const unsigned roff = 4u * (unsigned)att_base(g, a, b);
                const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
                const int kstart = (k0 <= k1) ? (k0 & ~3) : k1 + 1;
                const float e_ray = PAIRED ? A.E[cand * A.e_cs + ray] : 0.f;
                const float rho2 =
                    PAIRED ? A.rho[cand * A.sino_cs + (size_t)((a + g.nah) * g.nb + (g.nb - 1 - b))] : 0.f;
                Comp eb = comp_pick(ebj, j);
                for (int kc = kstart; kc <= k1; kc += kBandChunk) {
                    float4 av[kBandChunk / 4], bv[kBandChunk / 4];
#pragma unroll
                    for (int q = 0; q < kBandChunk / 4; ++q) {
                        const int k = kc + 4 * q;
                        const unsigned o = roff + 4u * att_row(g, k);
                        bv[q] = (k <= k1) ? buffer_ld4(rb, o, 0u) : z4;
                        av[q] = (PAIRED && k <= k1) ? buffer_ld4(ra, o, 0u) : z4;
                    }
                    float ov[4];
                    float epart = 0.f;
#pragma unroll
                    for (int q = 0; q < kBandChunk; ++q) {
                        const int k = kc + q;
                        ov[q & 3] = f4at(bv[q >> 2], q & 3);
                        if (k <= k1) {
                            float U, V;
                            sample_uv(Ub, Vb, tau_of(g, k), cs.x, cs.y, U, V);
                            const Tap t = make_tap<false>(U, V, nf, pitch, band);
                            if (t.mine) {
                                const float2 w = lerp2x2(lds2 + t.off, pitch, t.fu, t.fv);
                                const float base = A.accumulate ? ov[q & 3] : 0.f;
                                const float cv = g.dx * fmaf(rho, w.y, w.x);
                                if constexpr (PAIRED) {
                                    const float ri = inv_att(f4at(av[q >> 2], q & 3));
                                    const float ao = e_ray * ri;
                                    const float cv2 = g.dx * fmaf(rho2, w.y, w.x);
                                    epart = fmaf(cv2, ri, epart);
                                    ov[q & 3] = base + fmaf(-ao * ri, cv2, cv);
                                } else {
                                    ov[q & 3] = base + cv;
                                }
                            }
                        }
                        if ((q & 3) == 3 && k - 3 <= k1)
                            buffer_st4(rb, roff + 4u * att_row(g, k - 3), 0u, make_float4(ov[0], ov[1], ov[2], ov[3]));
                    }
                    if constexpr (PAIRED) kahan_add(eb, epart);
                }
                if constexpr (PAIRED) comp_put(ebj, j, eb);
            }
        }
    }
    if constexpr (!SINGLE) {
        // pass 2: every sample of the ray now holds att_bar (written by this thread): scan
#pragma unroll
        for (int j = 0; j < kMaxRpt; ++j) {
            if (j >= rpt) break;
            const int ray = band_ray(chunk, chunks, j);
            if (ray >= nrays) continue;
            const int a = ray / g.nb, b = ray - a * g.nb;
            // 16 samples (4 groups, one 16-byte access each) at a time: the chunk's loads are issued
            // before any of its stores; padding rows get 0
            const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(att, (unsigned)(4 * A.att_cs));
            const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(ab, (unsigned)(4 * A.att_cs));
            const unsigned roff = 4u * (unsigned)att_base(g, a, b);
            const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
            Comp P{0.f, 0.f};
            for (int kc = 0; kc < g.nt; kc += kBandChunk) {
                float4 av[kBandChunk / 4], bv[kBandChunk / 4];
#pragma unroll
                for (int q = 0; q < kBandChunk / 4; ++q) {
                    const int k = kc + 4 * q;
                    const unsigned o = roff + 4u * att_row(g, k);
                    av[q] = (k < g.nt) ? buffer_ld4(ra, o, 0u) : z4;
                    bv[q] = (k < g.nt) ? buffer_ld4(rb, o, 0u) : z4;
                }
                float ov[4];
#pragma unroll
                for (int q = 0; q < kBandChunk; ++q) {
                    const int k = kc + q;
                    ov[q & 3] = 0.f;
                    if (k < g.nt) {
                        const float Lbar = -f4at(av[q >> 2], q & 3) * f4at(bv[q >> 2], q & 3);
                        ov[q & 3] = g.dx * (fmaf(0.5f, Lbar, P.s) + P.e);
                        comp_add(P, Lbar);
                    }
                    if ((q & 3) == 3 && k - 3 < g.nt)
                        buffer_st4(rb, roff + 4u * att_row(g, k - 3), 0u, make_float4(ov[0], ov[1], ov[2], ov[3]));
                }
            }
            if constexpr (PAIRED) {
                float *eo = A.Ebar + cand * A.e_cs + ray;
                const float etot = (A.accumulate ? *eo : 0.f) + comp_value(ebj[j]);
                *eo = g.dx * (-A.E[cand * A.e_cs + ray] * etot);
            }
        }
    }
}

#ifndef BOAC_BODIES_ONLY
template <bool SINGLE, bool PAIRED>
__global__ __launch_bounds__(1024) void k_tail(DevGeom g, Bands bands, int rpt, int chunks, int C, TailArgs A) {
    extern __shared__ float lds[];
    k_tail_body<SINGLE, PAIRED>(blockIdx.x, lds, g, bands, rpt, chunks, C, A);
}
#endif

// Forward projection for few candidates (a grid of one-thread-per-ray workgroups would leave most of the
// GPU idle): each ray is split over kSplitLanes lanes of one wave, lane j taking the 16-sample chunks j,
// j + kSplitLanes, ... of the ray. A chunk is summed exactly as in k_fwd's single-stage path (same
// positions, same bilinear reads, FMAs in sample order), and the chunk sums are then added to the
// compensated total in chunk order after a shuffle, so every ray's result equals k_fwd's and
// k_fwd_pair's bit for bit. Single-stage images, n_samples <= 16 kSplitLanes kSplitCpl. In the likelihood
// a ray's first lane forms its terms, and the workgroup's sum is its partial.
constexpr int kSplitLanes = 8;
constexpr int kSplitCpl = 2;  // chunks per lane

#ifndef BOAC_BODIES_ONLY
// AHEAD: the first loads go out before the image is staged, and more of the image at a time (see the plan).
template <int MODE, bool PAIRED, bool AHEAD>
__global__ __launch_bounds__(256, AHEAD ? 1 : 6) void k_fwd_split(DevGeom g, Band band, int chunks, int C, FwdArgs A) {
    extern __shared__ float lds[];
    __shared__ float red[32];
    int cand, chunk;
    ray_block(blockIdx.x, chunks, C, cand, chunk);
    const int nrays = g.nah * g.nb;
    const int pitch = band.pitch;
    const float nf = (float)g.n;
    const int lane = threadIdx.x & (kSplitLanes - 1);
    const int ray = chunk * (blockDim.x / kSplitLanes) + threadIdx.x / kSplitLanes;
    const bool live = ray < nrays;
    constexpr int KC = 16, KG = KC / 4;
    const int a = live ? ray / g.nb : 0, b = live ? ray - a * g.nb : 0;
    const int opp = (a + g.nah) * g.nb + (g.nb - 1 - b);
    const float2 cs = g.trig[a];
    float Ub, Vb;
    ray_base(g, sigma_of(g, b), cs.x, cs.y, Ub, Vb);
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(A.att + cand * A.att_cs, (unsigned)(4 * A.att_cs));
    const unsigned roff = 4u * (unsigned)att_base(g, a, b);
    const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
    const int nck = (g.nt + KC - 1) / KC;
    // the kernel is one chain of memory round trips: the first chunk of att, exp(-T) and the counts are on
    // their way while the image is staged
    float4 v0[AHEAD ? KG : 1];
    const bool has0 = live && lane < nck;
    if constexpr (AHEAD)
#pragma unroll
        for (int q = 0; q < KG; ++q)
            v0[q] = (has0 && lane * KC + 4 * q < g.nt) ? buffer_ld4_stream(rs, roff, 4u * att_row(g, lane * KC + 4 * q)) : z4;
    const float e_ray = (PAIRED && live) ? A.E[cand * A.e_cs + ray] : 0.f;
    const float S = live ? fwd_meas<MODE>(A, ray) : 0.f;
    const float S2 = (PAIRED && live) ? fwd_meas<MODE>(A, opp) : 0.f;
    stage_whole<AHEAD ? 16 : 8>(A.img + cand * A.img_cs, g.n, band, lds);
    __syncthreads();

    float part[kSplitCpl], part2[kSplitCpl];
#pragma unroll
    for (int h = 0; h < kSplitCpl; ++h) {
        part[h] = part2[h] = 0.f;
        const int ck = lane + h * kSplitLanes;
        if (!live || ck >= nck) continue;
        const int k0 = ck * KC;
        float4 v[KG];
#pragma unroll
        for (int q = 0; q < KG; ++q)
            v[q] = (AHEAD && h == 0) ? v0[AHEAD ? q : 0]
                          : (k0 + 4 * q < g.nt) ? buffer_ld4_stream(rs, roff, 4u * att_row(g, k0 + 4 * q)) : z4;
        float tau = (float)k0 - g.cT;
        float p = 0.f, p2 = 0.f;
        // samples past the ray's end are masked, not branched over: the chunk's LDS reads overlap
        const unsigned bits = band_bits(k0, 0, g.nt - 1);
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            float U, V;
            sample_uv(Ub, Vb, tau, cs.x, cs.y, U, V);
            const float at = f4at(v[q >> 2], q & 3);
            const float w = bit_keep(bits, q, bilinear_whole(lds, U, V, nf, pitch));
            p = fmaf(at, w, p);
            if constexpr (PAIRED) p2 = fmaf(opposed_att(e_ray, at), w, p2);
            tau += 1.f;
        }
        part[h] = p;
        part2[h] = p2;
    }
    // the compensated total over the chunks in order (chunk ck is in lane ck % L, slot ck / L)
    const int base = (threadIdx.x & (kWave - 1)) & ~(kSplitLanes - 1);
    Comp c{0.f, 0.f}, c2{0.f, 0.f};
    for (int ck = 0; ck < nck; ++ck) {
        const int h = ck / kSplitLanes;
        const float mine = (h == 0) ? part[0] : part[kSplitCpl - 1];
        kahan_add(c, __shfl(mine, base + ck % kSplitLanes, kWave));
        if constexpr (PAIRED) {
            const float mine2 = (h == 0) ? part2[0] : part2[kSplitCpl - 1];
            kahan_add(c2, __shfl(mine2, base + ck % kSplitLanes, kWave));
        }
    }
    bool zero_proj = false;
    Comp nll{0.f, 0.f};
    if (live && lane == 0) {
        const float t0 = fwd_emit<MODE>(A, cand, ray, S, g.dx * comp_value(c), zero_proj);
        if constexpr (MODE == FWD_NLL) comp_add(nll, t0);
        if constexpr (PAIRED) {
            const float t1 = fwd_emit<MODE>(A, cand, opp, S2, g.dx * comp_value(c2), zero_proj);
            if constexpr (MODE == FWD_NLL) comp_add(nll, t1);
        }
    }
    if constexpr (MODE == FWD_NLL) {
        if (zero_proj && A.status) atomicOr(A.status + cand, 1u);
        const Comp r = block_reduce(nll, red);
        if (threadIdx.x == 0) A.partial[(size_t)cand * chunks + chunk] = make_float2(r.s, r.e);
    }
}
#endif

#ifndef BOAC_BODIES_ONLY
// ------------------------------------------------------------------ launchers
static dim3 ray_grid(const RayCfg &rc, int C) { return dim3((unsigned)(rc.chunks * C)); }

hipError_t launch_att(const DevGeom &g, const RayCfg &rc, const Bands &bands, const float *mu, float *att,
                      size_t img_cs, size_t att_cs, float *E, size_t e_cs, int C, hipStream_t st) {
    if (TaskRecorder *r = task_recorder()) {
        TaskRec t{};
        if (rc.block != kPersistThreads)
            return record_unsupported(r, "attenuation build planned with other than 1024 threads");
        t.kind = T_ATT;
        t.variant = rc.single ? 1 : 0;
        int up = 0;
        const int chunks = rc.single ? rc.chunks : att_band_chunks(g.na, g.nah, g.nb, rc.block * rc.rpt, up);
        t.u.att = {RayTask{g, bands, rc.rpt, chunks, C}, mu, att, img_cs, att_cs, E, e_cs, up};
        t.grid = t.items = chunks * C;
        t.lds = (unsigned)rc.lds;
        return record_task(r, t);
    }
    if (rc.single && rc.scan_passes > 0) {
        hipLaunchKernelGGL(k_att_scan, dim3((unsigned)(rc.scan_chunks * C)), dim3(256), rc.lds, st, g,
                           bands.band(0, g.n), rc.scan_passes, rc.scan_chunks, C, mu, att, img_cs, att_cs, E, e_cs);
        return hipGetLastError();
    }
    if (rc.single) {
        const int per = rc.att_block * rc.att_rpt, chunks = (g.nah * g.nb + per - 1) / per;
        hipLaunchKernelGGL(k_att<true>, dim3((unsigned)chunks * (unsigned)C), dim3(rc.att_block), rc.lds, st, g, bands,
                           rc.att_rpt, chunks, 0, C, mu, att, img_cs, att_cs, E, e_cs);
    } else {
        int up;
        const int chunks = att_band_chunks(g.na, g.nah, g.nb, rc.att_block * rc.att_rpt, up);
        hipLaunchKernelGGL(k_att<false>, dim3((unsigned)chunks * (unsigned)C), dim3(rc.att_block), rc.lds, st, g, bands, rc.att_rpt,
                           chunks, up, C, mu, att, img_cs, att_cs, E, e_cs);
    }
    return hipGetLastError();
}

template <int MODE, bool PAIRED>
static void fwd_mode(const DevGeom &g, const RayCfg &rc, const Bands &bands, const FwdArgs &a, int C,
                     hipStream_t st) {
    if (rc.split_chunks > 0 && (MODE != FWD_NLL || rc.split_nll)) {
        const dim3 grid((unsigned)(rc.split_chunks * C));
        if (rc.split_ahead)
            hipLaunchKernelGGL((k_fwd_split<MODE, PAIRED, true>), grid, dim3(256), rc.lds, st, g, bands.band(0, g.n),
                               rc.split_chunks, C, a);
        else
            hipLaunchKernelGGL((k_fwd_split<MODE, PAIRED, false>), grid, dim3(256), rc.lds, st, g, bands.band(0, g.n),
                               rc.split_chunks, C, a);
        return;
    }
    if (rc.pair && rc.single && a.img_comps == 1 && C >= 2)
        hipLaunchKernelGGL((k_fwd_pair<MODE, PAIRED>), dim3((unsigned)(rc.chunks * ((C + 1) / 2))), dim3(rc.block),
                           2 * rc.lds, st, g, bands, rc.rpt, rc.chunks, C, a);
    else if (rc.single)
        hipLaunchKernelGGL((k_fwd<MODE, true, PAIRED>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands,
                           rc.rpt, rc.chunks, C, a);
    else
        hipLaunchKernelGGL((k_fwd<MODE, false, PAIRED>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands,
                           rc.rpt, rc.chunks, C, a);
}

hipError_t launch_fwd(int mode, const DevGeom &g, const RayCfg &rc, const Bands &bands, const FwdArgs &a, int C,
                      hipStream_t st) {
    if (TaskRecorder *r = task_recorder()) {
        if (rc.block != kPersistThreads) return record_unsupported(r, "projection planned with other than 1024 threads");
        if (mode != FWD_NLL && rc.split_chunks > 0) return record_unsupported(r, "ray-split projection");
        TaskRec t{};
        const bool pair = rc.pair && rc.single && a.img_comps == 1 && C >= 2;
        t.kind = pair ? T_FWD_PAIR : T_FWD;
        t.variant = mode | (rc.single ? 4 : 0) | (a.E ? 8 : 0);
        t.u.fwd = {RayTask{g, bands, rc.rpt, rc.chunks, C}, a};
        t.grid = t.items = rc.chunks * (pair ? (C + 1) / 2 : C);
        t.lds = (unsigned)(pair ? 2 * rc.lds : rc.lds);
        return record_task(r, t);
    }
    const bool paired = a.E != nullptr;
    if (paired && g.nah * 2 != g.na) return hipErrorInvalidValue;
    if (rc.split_chunks > 0 && (!rc.single || a.img_comps != 1 || g.nt > 16 * kSplitLanes * kSplitCpl))
        return hipErrorInvalidValue;
    switch (mode) {
        case FWD_PROJ: paired ? fwd_mode<FWD_PROJ, true>(g, rc, bands, a, C, st)
                              : fwd_mode<FWD_PROJ, false>(g, rc, bands, a, C, st); break;
        case FWD_RATIO: paired ? fwd_mode<FWD_RATIO, true>(g, rc, bands, a, C, st)
                               : fwd_mode<FWD_RATIO, false>(g, rc, bands, a, C, st); break;
        case FWD_NLL: paired ? fwd_mode<FWD_NLL, true>(g, rc, bands, a, C, st)
                             : fwd_mode<FWD_NLL, false>(g, rc, bands, a, C, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_adj_sweep(const DevGeom &g, const RayCfg &rc, const Bands &bands, const SweepArgs &a, int C,
                            hipStream_t st) {
    if (TaskRecorder *r = task_recorder()) {
        if (rc.block != kPersistThreads) return record_unsupported(r, "reverse sweep planned with other than 1024 threads");
        TaskRec t{};
        t.kind = T_SWEEP;
        t.variant = (rc.single ? 1 : 0) | (a.E ? 2 : 0);
        t.u.sweep = {RayTask{g, bands, rc.rpt, rc.chunks, C}, a};
        t.grid = t.items = rc.chunks * C;
        t.lds = (unsigned)rc.lds;
        return record_task(r, t);
    }
    const bool paired = a.E != nullptr;
    if (paired != (g.nah != g.na) || (paired && (g.nah * 2 != g.na || !a.Ebar))) return hipErrorInvalidValue;
    if (paired && rc.single)
        hipLaunchKernelGGL((k_adj_sweep<true, true>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands, rc.rpt,
                           rc.chunks, C, a);
    else if (paired)
        hipLaunchKernelGGL((k_adj_sweep<false, true>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands, rc.rpt,
                           rc.chunks, C, a);
    else if (rc.single)
        hipLaunchKernelGGL((k_adj_sweep<true, false>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands, rc.rpt,
                           rc.chunks, C, a);
    else
        hipLaunchKernelGGL((k_adj_sweep<false, false>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands,
                           rc.rpt, rc.chunks, C, a);
    return hipGetLastError();
}

hipError_t launch_tail(const DevGeom &g, const RayCfg &rc, const Bands &bands, const TailArgs &a, int C,
                       hipStream_t st) {
    if (TaskRecorder *r = task_recorder()) {
        if (rc.block != kPersistThreads) return record_unsupported(r, "adjoint tail planned with other than 1024 threads");
        TaskRec t{};
        t.kind = T_TAIL;
        t.variant = (rc.single ? 1 : 0) | (a.E ? 2 : 0);
        t.u.tail = {RayTask{g, bands, rc.rpt, rc.chunks, C}, a};
        t.grid = t.items = rc.chunks * C;
        t.lds = (unsigned)rc.lds;
        return record_task(r, t);
    }
    const bool paired = a.E != nullptr;
    if (paired != (g.nah != g.na) || (paired && (g.nah * 2 != g.na || !a.Ebar))) return hipErrorInvalidValue;
    if (paired && rc.single)
        hipLaunchKernelGGL((k_tail<true, true>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands, rc.rpt,
                           rc.chunks, C, a);
    else if (paired)
        hipLaunchKernelGGL((k_tail<false, true>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands, rc.rpt,
                           rc.chunks, C, a);
    else if (rc.single)
        hipLaunchKernelGGL((k_tail<true, false>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands, rc.rpt,
                           rc.chunks, C, a);
    else
        hipLaunchKernelGGL((k_tail<false, false>), ray_grid(rc, C), dim3(rc.block), rc.lds, st, g, bands, rc.rpt,
                           rc.chunks, C, a);
    return hipGetLastError();
}

#endif  // BOAC_BODIES_ONLY

}  // namespace boac
