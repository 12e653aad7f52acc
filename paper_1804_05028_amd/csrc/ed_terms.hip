// Stored terms: the targets of a sector's off-diagonal terms, searched once.
//
// The representative search and the index lookup of a term depend on the
// basis alone, not on the couplings or the vector, and a sector's H.v is
// repeated many times (each Lanczos step, each call of a fit).  Where the
// table fits, ed_build_basis therefore searches every term once and keeps one
// 32-bit word per term,
//   word = class << ibits | row index of the target,
// where the class names the bond's orbit and the character of the element
// found (times the Fermi sign, for fermions); the coefficients of the classes
// (J/2 chi) are rewritten when the couplings change.  Terms without a target
// in the sector keep their class (their bond counts in the diagonal) and
// point at row dim, whose amplitude is zero; padding has a class of its own
// whose coefficients are zero.
//
// Rows are taken in slices of 64, one per lane.  A slice holds as many groups
// of four terms as its longest row needs, a group being 64 lanes x 4 words, so
// that a wave reads its words as one 1 KB load.  A row's terms are in bond
// order, as in the searching kernels, and summed by the same operations: both
// give the same bits.
//
// A sector whose table is too large to keep (40-site square: 142 GB) gets one
// for the duration of a long Lanczos call, in half of the free memory; where
// that holds the first slices only, the searching kernel does the other rows.
#include "ed_device.hpp"

#include <type_traits>
#include <utility>

namespace ed {

constexpr int kTermsThreads = 256;
constexpr int kTermsWaves = kTermsThreads / kWave;
constexpr int kMaxClasses = 1024;
constexpr int kNextStride = kTermsNextStride;   // a counter per 128-byte line


// ---------------------------------------------------------------------------
// building
// ---------------------------------------------------------------------------

// groups of four terms of every slice
__global__ void __launch_bounds__(256) k_terms_count(DevModel dm, const uint64_t *states, int64_t D, uint32_t *cnt)
{
    __shared__ uint64_t mask[kMaxBondWords * 64];
    const BondLds *bonds = (const BondLds *)(dm.blob + dm.off_bonds);
    for (int k = threadIdx.x; k < dm.nb; k += blockDim.x) mask[k] = bonds[k].mask;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t n_slices = (D + kWave - 1) / kWave;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t n_waves = (int64_t)gridDim.x * blockDim.x / kWave;
    for (int64_t sl = wave; sl < n_slices; sl += n_waves) {
        const int64_t i = sl * kWave + lane;
        int n = 0;
        if (i < D) {
            const uint64_t s = states[i] & kStateMask;
            for (int k = 0; k < dm.nb; ++k) {
                const uint64_t t = s & mask[k];
                n += (t != 0) & (t != mask[k]);
            }
        }
        for (int o = 32; o > 0; o >>= 1) n = max(n, __shfl_xor(n, o, 64));
        if (lane == 0) cnt[sl] = (uint32_t)(n + 3) / 4;
    }
}

// Searches every term.  A wave takes a slice, or, where there are few slices,
// every parts-th term of one.  As in k_apply, the index entry (without an
// index, the slot) of the next term is requested before the current one is
// resolved.  The index costs a third of the lines of hashed slots, since neighbouring rows share entries: 32-site
// square 15.3 -> 6.5 ms, 30-site complex sector 3.9 -> 2.1 ms; the 864-element
// group, bound by its search, 29.9 -> 27.8 ms.
template <typename AT, int NSC, bool FERMI>
__global__ void __launch_bounds__(1024) k_terms_fill(DevModel dm, DevBasis db, RepIndex ix, const uint64_t *off, uint32_t stride,
                                                     uint32_t *cnt, uint32_t *words, const uint16_t *chi_class,
                                                     const uint16_t *bond_orbit, int n_orb, int ibits, uint32_t pad,
                                                     int parts, int64_t n_slices)
{
    extern __shared__ __align__(16) char lds[];
    const Ctx<AT> c = stage<AT>(dm, lds);
    const int nb = dm.nb;
    const int64_t D = db.dim;
    const uint64_t smask = (1ull << db.slot_log2) - 1ull;
    const int lane = threadIdx.x & (kWave - 1);
    const int sshift = dm.is_complex ? 5 : 4;
    const int64_t n_units = n_slices * parts;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int64_t n_waves = (int64_t)gridDim.x * blockDim.x / kWave;
    for (int64_t unit = wave; unit < n_units; unit += n_waves) {
        const int64_t slice = unit / parts;
        const int part = (int)(unit % parts);
        const int64_t i = slice * kWave + lane;
        const bool row_ok = i < D;
        const uint64_t s = row_ok ? db.states[i] & kStateMask : 0ull;
        BondMask am;
        am.w0 = bond_word(c, s, 0, nb);
        am.w1 = nb > 64 ? bond_word(c, s, 1, nb) : 0ull;
        am.w2 = nb > 128 ? bond_word(c, s, 2, nb) : 0ull;
        am.w3 = nb > 192 ? bond_word(c, s, 3, nb) : 0ull;
        const int n_terms = row_ok ? __popcll(am.w0) + __popcll(am.w1) + __popcll(am.w2) + __popcll(am.w3) : 0;
        int most = n_terms;
        for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
        const int groups = (most + 3) / 4;
        if (off == nullptr && part == 0 && lane == 0) cnt[slice] = (uint32_t)groups;
        const uint64_t base = off ? off[slice] : (uint64_t)slice * stride;
        uint64_t r_nx = 0, sl_nx = 0;
        uint32_t cl_nx = 0, k_nx = 0;
        ulonglong2 q_nx = make_ulonglong2(0ull, 0ull);
        int done = 0;   // bonds taken off the mask
        auto request = [&](int t) {
            int bi = 0;
            for (; done <= t; ++done) bi = pop_bond(am);
            const uint64_t sp = s ^ c.bonds[bi].mask;
            uint32_t g;
            r_nx = rep_search<AT, NSC>(c, sp, g);
            uint32_t neg = 0;
            if constexpr (FERMI)
                neg = ((uint32_t)__popcll(s & c.between[bi]) & 1u) ^ fermi_parity<AT, NSC>(c, c.g_u[g], sp);
            cl_nx = (uint32_t)chi_class[neg ? dm.ng + g : g] * n_orb + bond_orbit[bi];
            if (ix.entries) {
                const uint32_t k = ix.rank[r_nx & ((1ull << ix.R) - 1ull)];
                const uint64_t pre = ((uint64_t)ix.top_rank[r_nx >> (c.N - c.m)] << ix.mid_bits) |
                                     ((r_nx >> ix.R) & ((1ull << ix.mid_bits) - 1ull));
                k_nx = k & (kWave - 1);
                q_nx = ix.entries[pre * ix.chunks + k / kWave];
            } else {
                sl_nx = slot_of_state(r_nx, db.slot_log2);
                q_nx = *(const ulonglong2 *)(db.slots + (sl_nx << sshift));
            }
        };
        if (part < n_terms) request(part);
        for (int t = part; t < 4 * groups; t += parts) {
            const uint64_t r = r_nx, home = sl_nx;
            const uint32_t cl = cl_nx, k = k_nx;
            uint64_t sl = sl_nx;
            ulonglong2 q = q_nx;
            if (t + parts < n_terms) request(t + parts);
            uint32_t word = pad;
            if (t < n_terms && ix.entries) {
                // representatives outside the sector have no bit
                const bool in = q.x >> k & 1ull;
                word = cl << ibits | (in ? (uint32_t)q.y + (uint32_t)__popcll(q.x & ((1ull << k) - 1ull)) : (uint32_t)D);
            } else if (t < n_terms) {
                while (q.x != kEmpty && (q.x & kStateMask) != r) {
                    sl = next_slot(sl, home, smask, sshift == 5 ? 2 : 3);
                    q = *(const ulonglong2 *)(db.slots + (sl << sshift));
                }
                word = cl << ibits | (q.x == kEmpty ? (uint32_t)D : (uint32_t)q.y);
            }
            words[((base + (uint64_t)(t >> 2)) * kWave + lane) * 4 + (t & 3)] = word;
        }
    }
}

// ---------------------------------------------------------------------------
// H.v
// ---------------------------------------------------------------------------

// coefficients of the classes, 1/sqrt of the divisors and, for fermions, the
// bonds: what an H.v of stored terms keeps in LDS
template <bool CPLX>
struct TermsLds {
    const double *cls, *rsqrt;
    const BondLds *bonds;
};

static size_t terms_lds_bytes(const ed_basis *b)
{
    return (size_t)b->terms.n_cls * (b->dm.is_complex ? 32 : 16) + (size_t)b->dm.n_div * 8 +
           (b->fermion ? (size_t)b->dm.nb * sizeof(BondLds) : 0);
}

template <bool CPLX, bool FERMI>
__device__ __forceinline__ TermsLds<CPLX> stage_terms(const DevModel &dm, const TermsDev &td, double *lds)
{
    const int n = td.n_cls * (CPLX ? 4 : 2);
    for (int k = threadIdx.x; k < n; k += blockDim.x) lds[k] = td.cls[k];
    const double *rs = (const double *)(dm.blob + dm.off_div) + dm.n_div;
    for (int k = threadIdx.x; k < dm.n_div; k += blockDim.x) lds[n + k] = rs[k];
    TermsLds<CPLX> t;
    t.cls = lds;
    t.rsqrt = lds + n;
    t.bonds = (const BondLds *)(lds + n + dm.n_div);
    if (FERMI) {
        const double *src = (const double *)(dm.blob + dm.off_bonds);
        for (int k = threadIdx.x; k < dm.nb * (int)(sizeof(BondLds) / 8); k += blockDim.x) lds[n + dm.n_div + k] = src[k];
    }
    __syncthreads();
    return t;
}

// the words of groups first .. first + kUnroll - 1; padding beyond the last
template <int U>
__device__ __forceinline__ void load_part(uint4 (&w)[U], const uint4 *p, int first, int groups, uint32_t none)
{
#pragma unroll
    for (int u = 0; u < U; ++u)
        w[u] = first + u < groups ? load_words(p + (size_t)(first + u) * kWave) : make_uint4(none, none, none, none);
}

// their terms, all gathers requested before the first is used; anti collects
// the Ising parts of their bonds
template <bool CPLX, int U, typename XS>
__device__ __forceinline__ void add_part(const TermsLds<CPLX> &tl, const uint4 (&w)[U], int first, int groups, int ibits, XS xs,
                                         double &ar, double &ai, double &anti)
{
    const uint32_t im = (1u << ibits) - 1u;
    typename Scalar<CPLX>::T v[U * 4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (first + u >= groups) break;   // uniform
        v[4 * u] = xs(w[u].x & im);
        v[4 * u + 1] = xs(w[u].y & im);
        v[4 * u + 2] = xs(w[u].z & im);
        v[4 * u + 3] = xs(w[u].w & im);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (first + u >= groups) break;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t cl = (k == 0 ? w[u].x : k == 1 ? w[u].y : k == 2 ? w[u].z : w[u].w) >> ibits;
            if constexpr (CPLX) {
                const double2 c = *(const double2 *)(tl.cls + 4 * cl);
                add_term<true>(ar, ai, c.x, c.y, v[4 * u + k].x, v[4 * u + k].y);
                anti += tl.cls[4 * cl + 2];
            } else {
                const double2 c = *(const double2 *)(tl.cls + 2 * cl);
                add_term<false>(ar, ai, c.x, 0.0, v[4 * u + k], 0.0);
                anti += c.y;
            }
        }
    }
}

template <bool CPLX, bool FERMI>
__device__ __forceinline__ double diagonal(const TermsLds<CPLX> &tl, int nb, uint64_t e, double anti, double jsq)
{
    if (!FERMI) return jsq - anti;
    const uint64_t s = e & kStateMask;
    double d = 0.0;
    for (int k = 0; k < nb; ++k) {
        const uint64_t bm = tl.bonds[k].mask;
        if ((s & bm) == bm) d += tl.bonds[k].jzhalf;
    }
    return d;
}

// y_i from the finished sums; returns Re(conj(x_i) y_i) in MODE 2
template <bool CPLX, int MODE>
__device__ __forceinline__ double finish_row(double rs, double ar, double ai, double d, typename Scalar<CPLX>::T xi,
                                             typename Scalar<CPLX>::T vp, const LzState &lz, typename Scalar<CPLX>::T *y)
{
    const double beta_prev = lz.beta_prev, inv = lz.inv, inv_prev = lz.inv_prev;
    double dot = 0.0;
    typename Scalar<CPLX>::T out;
    if constexpr (CPLX) {
        if (MODE == 2) {
            xi.x *= inv;
            xi.y *= inv;
            ar *= inv;
            ai *= inv;
        }
        out.x = fma(rs, ar, d * xi.x);
        out.y = fma(rs, ai, d * xi.y);
        if (MODE == 2) {
            out.x = fma(-beta_prev, inv_prev * vp.x, out.x);
            out.y = fma(-beta_prev, inv_prev * vp.y, out.y);
            dot = fma(xi.x, out.x, xi.y * out.y);
        }
    } else {
        if (MODE == 2) {
            xi *= inv;
            ar *= inv;
        }
        out = fma(rs, ar, d * xi);
        if (MODE == 2) {
            out = fma(-beta_prev, inv_prev * vp, out);
            dot = xi * out;
        }
    }
    *y = out;
    return dot;
}

// a slice's first words and its lane's row, requested together
template <bool CPLX, int MODE, int U>
struct TermsSlice {
    using T = typename Scalar<CPLX>::T;
    int64_t i;
    int groups;
    bool ok;
    const uint4 *p;
    uint4 w[U];
    uint64_t e;
    T xi, vp;
    __device__ __forceinline__ void request(const TermsDev &td, uint32_t none, int64_t slice, int lane, const uint64_t *states,
                                            int64_t D, const T *x, const T *vprev)
    {
        i = slice * kWave + lane;
        ok = i < D;
        groups = (int)td.cnt[slice];
        p = td.words + (td.off ? td.off[slice] : (uint64_t)slice * td.stride) * kWave + lane;
        load_part<U>(w, p, 0, groups, none);
        e = ok ? states[i] : 0ull;
        xi = T{};
        vp = T{};
        if (ok) {
            xi = x[i];
            if (MODE == 2) vp = vprev[i];
        }
    }
};

template <bool CPLX, int MODE, bool FERMI, int U, typename XS>
__device__ __forceinline__ double terms_row(const TermsLds<CPLX> &tl, const TermsDev &td, uint32_t none, int nb,
                                            TermsSlice<CPLX, MODE, U> &sl, XS xs, typename Scalar<CPLX>::T *y, const LzState &lz,
                                            double jsq)
{
    double ar = 0.0, ai = 0.0, anti = 0.0;
    // the words of the next groups are read while these are gathered
    uint4 nx[U];
    for (int g = 0; g < sl.groups; g += U) {
        load_part<U>(nx, sl.p, g + U, sl.groups, none);
        add_part<CPLX, U>(tl, sl.w, g, sl.groups, td.ibits, xs, ar, ai, anti);
#pragma unroll
        for (int u = 0; u < U; ++u) sl.w[u] = nx[u];
    }
    return sl.ok ? finish_row<CPLX, MODE>(tl.rsqrt[sl.e >> kNormShift], ar, ai, diagonal<CPLX, FERMI>(tl, nb, sl.e, anti, jsq),
                                          sl.xi, sl.vp, lz, y + sl.i)
                 : 0.0;
}

// H.v from the stored terms: a coalesced read of the words and a gather of
// scaled amplitudes, bound by the lines of 128 bytes that the gathers miss in
// L2 (random lines come at 55e9 per second here, from HBM and MALL alike).
// The rows are in ascending order and consecutive rows differ in their last
// bits, so that the targets of one bond lie close together too: on the 32-site
// square sector the 64 rows of a slice touch 0.57 lines per term and load
// instruction, 0.35 over all their terms, and 8192 consecutive rows 0.21
// (36-site triangular: 0.74, 0.51, 0.20), where hashed slots cost 1.04.
// chunks = 8 gives each XCD (blocks go round the XCDs in turn) one contiguous
// range of rows, which its L2 then shares.
//
// Lines are shared only while they stay in L2, so few rows should be in work
// at a time, and these should be neighbours.  Where the input exceeds the L2s,
// one block per compute unit runs (four waves with 32 gathers of each lane in
// flight; 2, 3, 5, 6 or 8 waves and 8 to 20 gathers were slower on one cluster
// or the other) and a wave takes the next slice of its XCD's range from a counter:
// with a fixed stride the waves drift apart and so do their rows.  32-site
// square 4.68 ms with eight blocks and a fixed stride, 3.91 with one, 3.05
// with the counter; 36-site triangular 5.20, 4.47, 3.46 ms.  The 1.4e6 rows of
// the 28-site square (11 MB) gain nothing: 157, 171, 179 us.
template <bool CPLX, int MODE, bool FERMI, bool COUNTED>
__global__ void __launch_bounds__(kTermsThreads)
    k_terms_apply(DevModel dm, TermsDev td, const uint64_t *__restrict__ states, int64_t D,
                  const typename Scalar<CPLX>::T *__restrict__ xs, const typename Scalar<CPLX>::T *__restrict__ x,
                  typename Scalar<CPLX>::T *__restrict__ y, const typename Scalar<CPLX>::T *__restrict__ vprev,
                  double *partials, LzStep step_of, double jsq, int chunks, unsigned int *next)
{
    using T = typename Scalar<CPLX>::T;
    extern __shared__ __align__(16) double lds_d[];
    constexpr int U = 8;   // groups in flight
    __shared__ double sh[kTermsWaves + 1];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t none = (uint32_t)(td.n_cls - 1) << td.ibits | (uint32_t)D;
    const int64_t n_slices = td.n_slices;
    const int64_t per = (n_slices + chunks - 1) / chunks;
    const int64_t first = per * (blockIdx.x % chunks);
    const int64_t last = min(first + per, n_slices);
    const int64_t step = (int64_t)(gridDim.x / chunks) * kTermsWaves;
    auto gather = [&](uint32_t j) { return *(const T *)((const char *)xs + (uint32_t)(j * (uint32_t)sizeof(T))); };
    TermsSlice<CPLX, MODE, U> sl;
    int64_t k = first + (int64_t)(blockIdx.x / chunks) * kTermsWaves + wave;
    // the first slice is on its way while the tables are staged: a short sector
    // is all latency
    if (!COUNTED && k < last) sl.request(td, none, k, lane, states, D, x, vprev);
    LzState lz{};
    if (MODE == 2 && !lz_begin(step_of, sh, lz)) return;
    const TermsLds<CPLX> tl = stage_terms<CPLX, FERMI>(dm, td, lds_d);
    if constexpr (COUNTED) {
        // the counter's last value is taken by every wave of the range in turn
        // beyond its end; k_pack and k_lz_update set it back to 0
        unsigned int *ctr = next + kNextStride * (blockIdx.x % chunks);
        unsigned int mine = lane == 0 ? atomicAdd(ctr, 1u) : 0u;
        while (true) {
            k = first + (int64_t)(unsigned int)__builtin_amdgcn_readfirstlane((int)mine);
            if (k >= last) return;
            mine = lane == 0 ? atomicAdd(ctr, 1u) : 0u;   // the one after, asked for early
            sl.request(td, none, k, lane, states, D, x, vprev);
            const double t = terms_row<CPLX, MODE, FERMI, U>(tl, td, none, dm.nb, sl, gather, y, lz, jsq);
            // which wave takes a slice varies from run to run: one sum per slice
            if (MODE == 2) {
                const double ws = wave_sum(t);
                if (lane == 0) partials[k] = ws;
            }
        }
    }
    double dot = 0.0;
    while (!COUNTED && k < last) {
        dot += terms_row<CPLX, MODE, FERMI, U>(tl, td, none, dm.nb, sl, gather, y, lz, jsq);
        k += step;
        if (k < last) sl.request(td, none, k, lane, states, D, x, vprev);
    }
    if (MODE == 2) {
        const double t = block_sum(dot, sh);
        if (threadIdx.x == 0) partials[blockIdx.x] = t;
    }
}

// the slices' <v, w> in kDotBlocks partial sums
__global__ void __launch_bounds__(kTermsThreads) k_terms_dots(const double *dots, int64_t n, double *partials, const LzState *lz)
{
    __shared__ double sh[kTermsWaves];
    if (lz->done) return;
    double a = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) a += dots[k];
    const double t = block_sum(a, sh);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// The same for sectors whose input fits LDS: every block scales all of x into
// LDS itself, so that one launch does the whole H.v and the gathers stay on
// the compute unit.  At 822 rows the call is one launch.
template <bool CPLX, bool FERMI>
__global__ void __launch_bounds__(kTermsThreads)
    k_terms_apply_small(DevModel dm, TermsDev td, const uint64_t *__restrict__ states, int64_t D,
                        const typename Scalar<CPLX>::T *__restrict__ x, typename Scalar<CPLX>::T *__restrict__ y, double jsq)
{
    using T = typename Scalar<CPLX>::T;
    extern __shared__ __align__(16) double lds_d[];
    constexpr int U = 8;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t n_slices = (D + kWave - 1) / kWave, slice = (int64_t)blockIdx.x * kTermsWaves + wave;
    const uint32_t none = (uint32_t)(td.n_cls - 1) << td.ibits | (uint32_t)D;
    TermsSlice<CPLX, 0, U> sl;
    if (slice < n_slices) sl.request(td, none, slice, lane, states, D, x, nullptr);
    T *xs = (T *)lds_d;
    const double *sq = (const double *)(dm.blob + dm.off_div);
    for (int k = threadIdx.x; k < (int)D; k += blockDim.x) {
        const double q = sq[states[k] >> kNormShift];
        T v = x[k];
        if constexpr (CPLX) {
            v.x *= q;
            v.y *= q;
        } else {
            v *= q;
        }
        xs[k] = v;
    }
    if (threadIdx.x == 0) xs[D] = T{};
    // the class table starts on a 16-byte boundary
    const TermsLds<CPLX> tl = stage_terms<CPLX, FERMI>(dm, td, lds_d + (((D + 1) * (CPLX ? 2 : 1) + 1) & ~(int64_t)1));
    auto gather = [&](uint32_t j) { return xs[j]; };
    if (slice < n_slices) terms_row<CPLX, 0, FERMI, U>(tl, td, none, dm.nb, sl, gather, y, LzState{}, jsq);
}

// blocks of a pass over all slices: a multiple of 8 (see chunks) where there
// are at least 8 blocks' worth; one per compute unit with the slice counter,
// else at most 8
int terms_grid(const ed_basis *b)
{
    const int64_t blocks = (b->terms.n_slices + kTermsWaves - 1) / kTermsWaves;
    if (blocks < 8) return (int)std::max<int64_t>(blocks, 1);
    return (int)std::min<int64_t>((blocks + 7) & ~7ll, (int64_t)(num_cus() * (b->terms.next ? 1 : 8) & ~7));
}

static int terms_chunks(const ed_basis *b) { return terms_grid(b) % 8 == 0 ? 8 : 1; }

template <bool CPLX, int MODE, bool FERMI>
static int launch_terms(const ed_basis *b, const void *x, void *y, const void *vprev, double *partials, const void *lz,
                        double jsq, hipStream_t st)
{
    using T = typename Scalar<CPLX>::T;
    const size_t lds = terms_lds_bytes(b);
    if (MODE == 0 && terms_small(b)) {
        const size_t xb = (((size_t)b->db.dim + 1) * sizeof(T) + 15) & ~(size_t)15;
        const int64_t slices = (b->db.dim + kWave - 1) / kWave;
        hipLaunchKernelGGL((k_terms_apply_small<CPLX, FERMI>), dim3((unsigned)((slices + kTermsWaves - 1) / kTermsWaves)),
                           dim3(kTermsThreads), xb + lds, st, b->dm, terms_dev(b), b->db.states, b->db.dim, (const T *)x,
                           (T *)y, jsq);
    } else {
        const LzStep ls = lz ? *(const LzStep *)lz : LzStep{};
#define ED_TERMS(COUNTED) \
    hipLaunchKernelGGL((k_terms_apply<CPLX, MODE, FERMI, COUNTED>), dim3(terms_grid(b)), dim3(kTermsThreads), lds, st, b->dm, \
                       terms_dev(b), b->db.states, b->db.dim, (const T *)b->terms.xs, (const T *)x, (T *)y, \
                       (const T *)vprev, partials, ls, jsq, terms_chunks(b), b->terms.next)
        if (b->terms.next) ED_TERMS(true);
        else ED_TERMS(false);
#undef ED_TERMS
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(ED_ERR_HIP, "H.v launch failed: %s", hipGetErrorString(e));
    return ED_OK;
}

template <int MODE>
static int terms_dispatch(const ed_basis *b, const void *x, void *y, const void *vprev, double *partials, const void *lz,
                          double jsq, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (b->fermion)
        return b->dm.is_complex ? launch_terms<true, MODE, true>(b, x, y, vprev, partials, lz, jsq, st)
                                : launch_terms<false, MODE, true>(b, x, y, vprev, partials, lz, jsq, st);
    return b->dm.is_complex ? launch_terms<true, MODE, false>(b, x, y, vprev, partials, lz, jsq, st)
                            : launch_terms<false, MODE, false>(b, x, y, vprev, partials, lz, jsq, st);
}

// y = H x; the scaled x is in terms.xs unless the sector is small
int terms_apply(const ed_basis *b, const void *x, void *y, double jsq, void *stream)
{
    return terms_dispatch<0>(b, x, y, nullptr, nullptr, nullptr, jsq, stream);
}

int sum_slices(const double *dots, int64_t n, double *partials, const void *lz, void *stream)
{
    hipLaunchKernelGGL(k_terms_dots, dim3(kDotBlocks), dim3(kTermsThreads), 0, (hipStream_t)stream, dots, n, partials,
                       (const LzState *)lz);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(ED_ERR_HIP, "slice sums: %s", hipGetErrorString(e));
    return ED_OK;
}

int terms_lanczos_apply(const ed_basis *b, const void *v, void *w, const void *vprev, double *partials, const void *lz,
                        double jsq, void *stream)
{
    return terms_dispatch<2>(b, v, w, vprev, partials, lz, jsq, stream);
}

// ---------------------------------------------------------------------------
// Lanczos of a sector whose scaled vector fits LDS (terms_small): one block
// does the whole iteration, its vectors in registers, two block sums per step
// in place of kernels.  The diagonal stays in a register, and the words of as
// many slices as fit the rest of LDS stay there, 16 bits each (where class and
// row fit them), instead of coming from L2 through one compute unit in every
// step.  A step is then bound by its reads of LDS.  20-site square, J1-J2,
// 1321 rows, 24 steps: 182 us (249 with the words read from L2, a sum by one
// thread and three barriers per total), 4x4 square 85 us (120); two kernels per
// step take 31 us each.
// ---------------------------------------------------------------------------
constexpr int kSmallThreads = 1024;
constexpr int kSmallSlices = 64;

// the wave's sum, in lane 63
__device__ __forceinline__ double wave_sum_last(double v)
{
    // in registers, where __shfl_xor goes through LDS: row_shr 1, 2, 4, 8 within 16 lanes, then row_bcast 15 and 31
    auto from = [&](auto ctrl, auto rows) {
        const long long b = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)b, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        v += __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    };
    using all = std::integral_constant<int, 0xf>;
    from(std::integral_constant<int, 0x111>{}, all{});
    from(std::integral_constant<int, 0x112>{}, all{});
    from(std::integral_constant<int, 0x114>{}, all{});
    from(std::integral_constant<int, 0x118>{}, all{});
    from(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
    from(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
    return v;
}

template <bool CPLX, bool FERMI>
__global__ void __launch_bounds__(kSmallThreads)
    k_terms_lanczos_small(DevModel dm, TermsDev td, const uint64_t *__restrict__ states, int D,
                          const typename Scalar<CPLX>::T *__restrict__ v0, int n_steps, double tol, double *alpha, double *beta,
                          LzState *state, typename Scalar<CPLX>::T *psi0, const double *svec, double jsq, int room, int words_at)
{
    using T = typename Scalar<CPLX>::T;
    constexpr int R = CPLX ? 2 : 4;   // rows of a thread (terms_small)
    constexpr int U = CPLX ? 2 : 3, H = 2;
    extern __shared__ __align__(16) double lds_d[];
    constexpr int kWaves = kSmallThreads / kWave;
    __shared__ __align__(16) double sh[2][kWaves];
    __shared__ int first[kSmallSlices + 1];   // groups before every slice
    T *xs = (T *)lds_d;
    uint2 *kept = (uint2 *)(lds_d + words_at);   // room groups of 64 x 4 words of 16 bits
    const TermsLds<CPLX> tl = stage_terms<CPLX, FERMI>(dm, td, lds_d + ((((size_t)D + 1) * (CPLX ? 2 : 1) + 1) & ~(size_t)1));
    double *sqrts = lds_d + words_at - dm.n_div;
    for (int k = threadIdx.x; k < dm.n_div; k += kSmallThreads) sqrts[k] = ((const double *)(dm.blob + dm.off_div))[k];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t none = (uint32_t)(td.n_cls - 1) << td.ibits | (uint32_t)D;
    auto gather = [&](uint32_t j) { return xs[j]; };
    auto uniform = [](int n) { return __builtin_amdgcn_readfirstlane(n); };
    // sums over the block in a fixed order, one barrier each: the two buffers
    // take turns
    int turn = 0;
    auto total = [&](double a) {
        const double t = wave_sum_last(a);
        double *part = sh[turn];
        turn ^= 1;
        if (lane == kWave - 1) part[threadIdx.x / kWave] = t;
        __syncthreads();
        double p[kWaves];
#pragma unroll
        for (int k = 0; k < kWaves; ++k) p[k] = part[k];
#pragma unroll
        for (int o = 1; o < kWaves; o *= 2)
#pragma unroll
            for (int k = 0; k < kWaves; k += 2 * o) p[k] += p[k + o];
        return p[0];
    };
    auto times = [](T v, double f) {
        if constexpr (CPLX)
            return make_double2(v.x * f, v.y * f);
        else
            return v * f;
    };
    auto norm2 = [](T v) {
        if constexpr (CPLX)
            return v.x * v.x + v.y * v.y;
        else
            return v * v;
    };
    if (threadIdx.x < kSmallSlices) {
        int n = threadIdx.x < td.n_slices ? (int)td.cnt[threadIdx.x] : 0;
        for (int o = 1; o < kSmallSlices; o *= 2) {
            const int m = __shfl_up(n, o, 64);
            if (lane >= o) n += m;
        }
        first[threadIdx.x + 1] = n;
        if (threadIdx.x == 0) first[0] = 0;
    }
    __syncthreads();
    const int ib = 32 - __clz(D);   // bits of a row or D
    const uint32_t im = (1u << td.ibits) - 1u;
    const uint32_t none16 = ((uint32_t)(td.n_cls - 1) << ib | (uint32_t)D) * 0x10001u;
    const bool one_class = td.n_cls == 2;   // and the padding
    const double c0 = tl.cls[0];
    T v[R], prev[R], psi[R];
    uint32_t div = 0;   // the rows' stabiliser sizes, 8 bits each
    double diag[R], acc = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = threadIdx.x + r * kSmallThreads;
        v[r] = prev[r] = psi[r] = T{};
        uint64_t e = 0;
        if (i < D) {
            e = states[i];
            div |= (uint32_t)(e >> kNormShift) << 8 * r;
            v[r] = v0[i];
        }
        acc += norm2(v[r]);
        diag[r] = 0.0;
        if (i - lane < D) {   // uniform: the wave's slice
            const int sl = uniform(i / kWave), from = uniform(first[sl]), groups = uniform(first[sl + 1]) - from;
            const uint4 *p = td.words + (td.off ? td.off[sl] : (uint64_t)sl * td.stride) * kWave + lane;
            double anti = 0.0;
            auto half = [&](uint32_t w) {
                anti += tl.cls[(CPLX ? 4 : 2) * (w >> td.ibits) + (CPLX ? 2 : 1)];
                return (w >> td.ibits << ib) | (w & im);
            };
            for (int g = 0; g < groups; ++g) {
                const uint4 w = load_words(p + (size_t)g * kWave);
                const uint32_t a = half(w.x), b = half(w.y), c = half(w.z), d = half(w.w);
                if (from + groups <= room) kept[(from + g) * kWave + lane] = make_uint2(a | b << 16, c | d << 16);
            }
            diag[r] = diagonal<CPLX, FERMI>(tl, dm.nb, e, anti, jsq);
        }
    }
    const double n2 = total(acc);
    LzState st{};
    st.inv = st.inv_prev = 1.0;   // v and prev are kept normalised
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = times(v[r], n2 > 0.0 ? 1.0 / sqrt(n2) : 0.0);
    if (threadIdx.x == 0) xs[D] = T{};
    double keep_a = 0.0, keep_b = 0.0;
    while (!st.done) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = threadIdx.x + r * kSmallThreads;
            if (i < D) xs[i] = times(v[r], sqrts[div >> 8 * r & 255u]);
        }
        __syncthreads();
        T w[R];
        double dot = 0.0;
        const double sj = psi0 ? svec[st.j] : 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) w[r] = T{};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = threadIdx.x + r * kSmallThreads;
            if (i - lane >= D) break;   // uniform: the wave's slice
            const int sl = uniform(i / kWave), from = uniform(first[sl]), groups = uniform(first[sl + 1]) - from;
            double ar = 0.0, ai = 0.0, anti = 0.0;
            if (from + groups <= room) {
                const uint2 *p = kept + from * kWave + lane;
                const uint32_t hm = (1u << ib) - 1u;
                for (int g = 0; g < groups; g += H) {
                    uint2 q[H];
                    T x[4 * H];
#pragma unroll
                    for (int u = 0; u < H; ++u)
                        if (g + u < groups) q[u] = p[(g + u) * kWave];
                        else q[u] = make_uint2(none16, none16);
                    auto each = [&](auto &&f) {
#pragma unroll
                        for (int u = 0; u < H; ++u) {
                            f(4 * u, q[u].x & 0xffffu);
                            f(4 * u + 1, q[u].x >> 16);
                            f(4 * u + 2, q[u].y & 0xffffu);
                            f(4 * u + 3, q[u].y >> 16);
                        }
                    };
                    each([&](int k, uint32_t h) { x[k] = xs[h & hm]; });
                    each([&](int k, uint32_t h) {
                        if constexpr (CPLX) {
                            const double2 c = *(const double2 *)(tl.cls + 4 * (h >> ib));
                            add_term<true>(ar, ai, c.x, c.y, x[k].x, x[k].y);
                        } else {
                            add_term<false>(ar, ai, one_class ? (h >> ib ? 0.0 : c0) : tl.cls[2 * (h >> ib)], 0.0, x[k], 0.0);
                        }
                    });
                }
            } else {
                const uint4 *p = td.words + (td.off ? td.off[sl] : (uint64_t)sl * td.stride) * kWave + lane;
                uint4 q[U], nx[U];
                load_part<U>(q, p, 0, groups, none);
                for (int g = 0; g < groups; g += U) {
                    load_part<U>(nx, p, g + U, groups, none);
                    add_part<CPLX, U>(tl, q, g, groups, td.ibits, gather, ar, ai, anti);
#pragma unroll
                    for (int u = 0; u < U; ++u) q[u] = nx[u];
                }
            }
            if (i < D) dot += finish_row<CPLX, 2>(tl.rsqrt[div >> 8 * r & 255u], ar, ai, diag[r], v[r], prev[r], st, &w[r]);
        }
        const double a = total(dot);
        acc = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (CPLX) {
                w[r].x -= a * v[r].x;
                w[r].y -= a * v[r].y;
                psi[r].x += sj * v[r].x;
                psi[r].y += sj * v[r].y;
            } else {
                w[r] -= a * v[r];
                psi[r] += sj * v[r];
            }
            acc += norm2(w[r]);
        }
        const double b = sqrt(total(acc));
        // coefficients are kept, not stored in every step: a barrier would wait
        if (threadIdx.x == (st.j & (kSmallThreads - 1))) {
            keep_a = a;
            keep_b = b;
        }
        st.scale = fmax(st.scale, fmax(fabs(a), b));
        st.j += 1;
        st.done = b <= tol * st.scale || st.j >= n_steps;
        if (st.done || (st.j & (kSmallThreads - 1)) == 0) {
            const int from = (st.j - 1) & ~(kSmallThreads - 1);
            if (from + (int)threadIdx.x < st.j) {
                alpha[from + threadIdx.x] = keep_a;
                beta[from + threadIdx.x] = keep_b;
            }
        }
        st.beta_prev = b;
        const double inv = st.done ? 0.0 : 1.0 / b;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            prev[r] = v[r];
            v[r] = times(w[r], inv);
        }
    }
    if (threadIdx.x < 2) state[threadIdx.x] = st;
    if (psi0) {
        acc = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) acc += norm2(psi[r]);
        const double t = total(acc);
        const double f = t > 0.0 ? 1.0 / sqrt(t) : 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = threadIdx.x + r * kSmallThreads;
            if (i < D) psi0[i] = times(psi[r], f);
        }
    }
}

// the whole iteration (with psi0: its second pass) in one launch
int terms_lanczos_small(const ed_basis *b, const void *v0, int n_steps, double tol, double *alpha, double *beta, void *state,
                        void *psi0, const double *svec, double jsq, void *stream)
{
    const bool c = b->dm.is_complex;
    const size_t tables = (((((size_t)b->db.dim + 1) * (c ? 16 : 8) + 15) & ~(size_t)15) + terms_lds_bytes(b) + 7 +
                           (size_t)b->dm.n_div * 8) & ~(size_t)7;
    // groups of words kept in LDS (512 bytes each), beside a few hundred static bytes
    int cbits = 1, ib = 1;
    while ((1 << cbits) < b->terms.n_cls) ++cbits;
    while ((1ll << ib) <= b->db.dim) ++ib;
    const size_t limit = lds_limit() - 1024;
    const int64_t most = (int64_t)b->terms.n_slices * ((b->dm.nb + 3) / 4);
    const int room = cbits + ib > 16 || limit < tables ? 0 : (int)std::min<int64_t>((int64_t)(limit - tables) / 512, most);
    const size_t lds = tables + (size_t)room * 512;
#define ED_SMALL(C, F) \
    hipLaunchKernelGGL((k_terms_lanczos_small<C, F>), dim3(1), dim3(kSmallThreads), lds, (hipStream_t)stream, b->dm, \
                       terms_dev(b), b->db.states, (int)b->db.dim, (const Scalar<C>::T *)v0, n_steps, tol, alpha, beta, \
                       (LzState *)state, (Scalar<C>::T *)psi0, svec, jsq, room, (int)(tables / 8))
    if (c) {
        if (b->fermion) ED_SMALL(true, true);
        else ED_SMALL(true, false);
    } else {
        if (b->fermion) ED_SMALL(false, true);
        else ED_SMALL(false, false);
    }
#undef ED_SMALL
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(ED_ERR_HIP, "Lanczos launch failed: %s", hipGetErrorString(e));
    return ED_OK;
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------

// {sqrt(n) x, sqrt(n) gy} of every row, zero behind the last
template <bool CPLX>
__global__ void k_terms_pair(const typename Scalar<CPLX>::T *x, const typename Scalar<CPLX>::T *gy, const uint64_t *states,
                             const double *sqrts, double *pair, int64_t D)
{
    constexpr int W = CPLX ? 2 : 1;
    const double *xd = (const double *)x, *gd = (const double *)gy;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j <= D; j += (int64_t)gridDim.x * blockDim.x) {
        const double sq = j < D ? sqrts[states[j] >> kNormShift] : 0.0;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            pair[(2 * j) * W + k] = j < D ? xd[j * W + k] * sq : 0.0;
            pair[(2 * j + 1) * W + k] = j < D ? gd[j * W + k] * sq : 0.0;
        }
    }
}

// f(0), ..., f(N - 1), each with its number as a type: arrays indexed by it
// stay in registers
template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// Per-bond adjoint sums, the targets read from the stored terms; FUSED: gx =
// H gy in the same pass, x_j and gy_j from one read of the pair array.  All
// lanes visit a bond together; a lane's word is the one at its count of
// antiparallel bonds so far.  kAhead bonds are read ahead, so that twice as
// many dependent reads of a lane are two latencies.
// NB bounds the bonds: up to 128 have a register each in every lane for their
// sum, added across lanes once at the end; more (NB = 0) are added across the
// wave bond by bond and kept by lane b % 64.  The order is fixed either way.
// 32-site square, 64 bonds: 5.9 ms with a sum across the wave per bond and four
// bonds ahead, 5.4 with this; 24-site square 38 -> 25 us.
template <bool CPLX, bool FUSED, int NB>
__global__ void __launch_bounds__(kTermsThreads)
    k_terms_backward(DevModel dm, TermsDev td, const uint64_t *__restrict__ states, int64_t D,
                     const double *__restrict__ src, const typename Scalar<CPLX>::T *__restrict__ x,
                     const typename Scalar<CPLX>::T *__restrict__ gy, double *partials, double *__restrict__ gx, double jsq,
                     int chunks)
{
    constexpr int W = CPLX ? 2 : 1;
    constexpr int kAhead = 8;
    constexpr int V = FUSED ? 2 * W : W;   // doubles per target
    extern __shared__ __align__(16) double lds_d[];
    // characters of the classes, 1/sqrt of the divisors, bonds; the block's
    // sums take their place at the end
    double *chi = lds_d, *rsqrt = lds_d + td.n_cls * W;
    BondLds *bonds = (BondLds *)(rsqrt + dm.n_div);
    const int nb = dm.nb;
    for (int k = threadIdx.x; k < td.n_cls * W; k += blockDim.x) chi[k] = td.cls_chi[k];
    {
        const double *rs = (const double *)(dm.blob + dm.off_div) + dm.n_div;
        for (int k = threadIdx.x; k < dm.n_div; k += blockDim.x) rsqrt[k] = rs[k];
        const double *bs = (const double *)(dm.blob + dm.off_bonds);
        for (int k = threadIdx.x; k < nb * (int)(sizeof(BondLds) / 8); k += blockDim.x) ((double *)bonds)[k] = bs[k];
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t im = (1u << td.ibits) - 1u;
    const int64_t n_slices = (D + kWave - 1) / kWave;
    const int64_t per = (n_slices + chunks - 1) / chunks;
    const int64_t first = per * (blockIdx.x % chunks);
    const int64_t last = min(first + per, n_slices);
    const int64_t step = (int64_t)(gridDim.x / chunks) * kTermsWaves;
    double tot = 0.0;
    double acc[NB > 0 ? NB : 4];   // NB = 0: bonds b of lane b % 64, 64 apart
#pragma unroll
    for (int b = 0; b < (NB > 0 ? NB : 4); ++b) acc[b] = 0.0;
    for (int64_t sl = first + (int64_t)(blockIdx.x / chunks) * kTermsWaves + wave; sl < last; sl += step) {
        const int64_t i = sl * kWave + lane;
        const bool valid = i < D;
        const uint32_t *p = (const uint32_t *)(td.words + (td.off ? td.off[sl] : (uint64_t)sl * td.stride) * kWave) + lane * 4;
        uint64_t s = 0;
        double rs_i = 0.0, gx_r = 0.0, g_r = 0.0, g_i = 0.0;
        if (valid) {
            const uint64_t e = states[i];
            s = e & kStateMask;
            rs_i = rsqrt[e >> kNormShift];
            if (CPLX) {
                const double2 gv = *(const double2 *)&gy[i];
                const double2 xv = *(const double2 *)&x[i];
                g_r = gv.x;
                g_i = gv.y;
                gx_r = fma(gv.x, xv.x, gv.y * xv.y);
            } else {
                g_r = *(const double *)&gy[i];
                gx_r = g_r * *(const double *)&x[i];
            }
        }
        tot += gx_r;
        double anti_sum = 0.0, ar = 0.0, ai = 0.0;
        int pos = 0;
        // kAhead bonds from b0; put(k, c) takes the contribution of bond b0 + k,
        // k a compile-time number
        auto bonds_from = [&](int b0, auto put) {
            bool anti[kAhead];
            uint32_t word[kAhead];
            double v[kAhead][V];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const int b = b0 + k;
                anti[k] = false;
                word[k] = 0;
                if (b < nb) {
                    const uint64_t bm = bonds[b].mask, t = s & bm;
                    anti[k] = valid && t != 0 && t != bm;
                }
                if (anti[k]) {
                    word[k] = p[(size_t)(pos >> 2) * (kWave * 4) + (pos & 3)];
                    ++pos;
                }
            }
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                for (int m = 0; m < V; ++m) v[k][m] = 0.0;
                if (anti[k]) {
                    const double *q = src + (size_t)(word[k] & im) * V;
                    if constexpr (V == 1) {
                        v[k][0] = *q;
                    } else {
#pragma unroll
                        for (int m = 0; m < V; m += 2) {
                            const double2 a = *(const double2 *)(q + m);
                            v[k][m] = a.x;
                            v[k][m + 1] = a.y;
                        }
                    }
                }
            }
            static_for<kAhead>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                const int b = b0 + k;
                if (b >= nb) return;   // uniform
                double contrib = 0.0;
                if (anti[k]) {
                    const uint32_t cl = word[k] >> td.ibits;
                    const double cr = chi[cl * W], ci = CPLX ? chi[cl * W + W - 1] : 0.0;
                    contrib = -0.5 * gx_r;
                    // a dropped term (row D) adds nothing, also not to a sum that is not finite
                    if ((word[k] & im) < (uint32_t)D)
                        contrib = fma(0.5 * rs_i, adjoint_term<CPLX>(cr, ci, v[k][0], CPLX ? v[k][W - 1] : 0.0, g_r, g_i), contrib);
                    if (FUSED) {
                        const double jh = bonds[b].jhalf;
                        anti_sum += bonds[b].jzhalf;
                        add_term<CPLX>(ar, ai, jh * cr, jh * ci, v[k][FUSED ? W : 0], CPLX ? v[k][V - 1] : 0.0);
                    }
                }
                put(kc, contrib);
            });
        };
        if constexpr (NB > 0) {
            static_for<NB / kAhead>([&](auto bc) {
                constexpr int b0 = decltype(bc)::value * kAhead;
                if (b0 >= nb) return;
                bonds_from(b0, [&](auto kc, double c) { acc[b0 + decltype(kc)::value] += c; });
            });
        } else {
            for (int b0 = 0; b0 < nb; b0 += kAhead)
                bonds_from(b0, [&](auto kc, double c) {
                    const int b = b0 + decltype(kc)::value;
                    const double wsum = wave_sum(c);
                    if (lane == (b & (kWave - 1))) {
                        const int q = b >> 6;
                        if (q == 0) acc[0] += wsum;
                        else if (q == 1) acc[1] += wsum;
                        else if (q == 2) acc[2] += wsum;
                        else acc[3] += wsum;
                    }
                });
        }
        if (FUSED && valid) {
            const double d = jsq - anti_sum;
            if (CPLX) {
                double2 out;
                out.x = fma(rs_i, ar, d * g_r);
                out.y = fma(rs_i, ai, d * g_i);
                *(double2 *)&gx[2 * i] = out;
            } else {
                gx[i] = fma(rs_i, ar, d * g_r);
            }
        }
    }
    __syncthreads();
    double *red = lds_d;   // [waves][nb + 1]
    const int w1 = nb + 1;
    if constexpr (NB > 0) {
        static_for<NB>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            if (b >= nb) return;
            const double t = wave_sum(acc[b]);
            if (lane == 0) red[wave * w1 + b] = t;
        });
    } else {
        for (int b = lane; b < nb; b += kWave) {
            const int q = b >> 6;
            red[wave * w1 + b] = q == 0 ? acc[0] : q == 1 ? acc[1] : q == 2 ? acc[2] : acc[3];
        }
    }
    const double t = wave_sum(tot);
    if (lane == 0) red[wave * w1 + nb] = t;
    __syncthreads();
    for (int b = threadIdx.x; b < w1; b += blockDim.x) {
        double sum = 0.0;
        for (int w = 0; w < kTermsWaves; ++w) sum += red[w * w1 + b];
        partials[(size_t)blockIdx.x * w1 + b] = sum;
    }
}

// per-bond sums (and gx = H gy if given).  Without gx the scaled x is in
// terms.xs.  The partial sums live in scratch if it is given.
int terms_backward(const ed_basis *bc, const void *x, const void *gy, void *gx, double *gJ_host, double *scratch,
                   size_t scratch_doubles, double jsq, void *stream)
{
    ed_basis *b = const_cast<ed_basis *>(bc);
    hipStream_t st = (hipStream_t)stream;
    const int nb = b->t.nb, W = b->dm.is_complex ? 2 : 1;
    const int64_t D = b->db.dim;
    // as many blocks per compute unit as the bonds' registers leave room for,
    // each of which leaves a row of partial sums, and slices at a fixed stride:
    // the sums are the same on every run
    const int per_cu = nb <= 64 ? 2 : nb <= 128 ? 1 : 4;
    int64_t blocks = ((D + kWave - 1) / kWave + kTermsWaves - 1) / kTermsWaves;
    if (blocks >= 8) blocks = std::min<int64_t>((blocks + 7) & ~7ll, (int64_t)(num_cus() * per_cu & ~7));
    const int grid = (int)blocks, chunks = grid % 8 == 0 ? 8 : 1;
    const size_t n_part = (size_t)grid * (nb + 1);
    if (gx && !b->terms.pair) {
        void *p = nullptr;
        const size_t bytes = ((size_t)D + 1) * 16 * W;
        if (hipMalloc(&p, bytes) != hipSuccess) {   // the caller frees the table
            (void)hipGetLastError();
            return set_error(ED_ERR_OOM, "adjoint pairs (%zu bytes)", bytes);
        }
        b->terms.pair = (double *)p;
        b->device_bytes += (int64_t)bytes;
        b->terms.bytes += (int64_t)bytes;
    }
    double *partials = scratch;
    if (scratch && n_part + (size_t)(nb + 1) > scratch_doubles)
        return set_error(ED_ERR_UNSUPPORTED, "adjoint partials of %zu doubles exceed the %zu-double scratch array",
                         n_part + (size_t)(nb + 1), scratch_doubles);
    if (!scratch) {   // kept with the terms: the grid never changes
        if (!b->terms.adj) {
            const size_t bytes = (n_part + nb + 1) * 8;
            if (hipMalloc((void **)&b->terms.adj, bytes) != hipSuccess) {
                (void)hipGetLastError();
                b->terms.adj = nullptr;
                return set_error(ED_ERR_OOM, "adjoint partials");
            }
            b->device_bytes += (int64_t)bytes;
            b->terms.bytes += (int64_t)bytes;
        }
        partials = b->terms.adj;
    }
    double *out = partials + n_part;
    const size_t lds = std::max((size_t)b->terms.n_cls * W * 8 + (size_t)b->dm.n_div * 8 + (size_t)nb * sizeof(BondLds),
                                (size_t)kTermsWaves * (nb + 1) * 8);
    const double *sq = (const double *)(b->dm.blob + b->dm.off_div);
    const dim3 pgrid((unsigned)std::min<int64_t>((D + 256) / 256, (int64_t)num_cus() * 16));
#define ED_BACK(C, F) \
    do { \
        if (nb <= 64) ED_BACK_NB(C, F, 64); \
        else if (nb <= 128) ED_BACK_NB(C, F, 128); \
        else ED_BACK_NB(C, F, 0); \
    } while (0)
#define ED_BACK_NB(C, F, NB) \
    hipLaunchKernelGGL((k_terms_backward<C, F, NB>), dim3(grid), dim3(kTermsThreads), lds, st, b->dm, terms_dev(b), b->db.states, \
                       D, (const double *)(F ? b->terms.pair : b->terms.xs), (const Scalar<C>::T *)x, \
                       (const Scalar<C>::T *)gy, partials, (double *)gx, jsq, chunks)
    if (b->dm.is_complex) {
        if (gx) {
            hipLaunchKernelGGL(k_terms_pair<true>, pgrid, dim3(256), 0, st, (const double2 *)x, (const double2 *)gy,
                               b->db.states, sq, b->terms.pair, D);
            ED_BACK(true, true);
        } else {
            ED_BACK(true, false);
        }
    } else {
        if (gx) {
            hipLaunchKernelGGL(k_terms_pair<false>, pgrid, dim3(256), 0, st, (const double *)x, (const double *)gy,
                               b->db.states, sq, b->terms.pair, D);
            ED_BACK(false, true);
        } else {
            ED_BACK(false, false);
        }
    }
#undef ED_BACK
#undef ED_BACK_NB
    int rc = sum_partials_cols(partials, grid, nb + 1, out, stream);
    double h[kMaxBondWords * 64 + 1];
    hipError_t e = rc ? hipSuccess : hipMemcpyAsync(h, out, (size_t)(nb + 1) * 8, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (rc) return rc;
    if (e != hipSuccess) return set_error(ED_ERR_HIP, "adjoint failed: %s", hipGetErrorString(e));
    for (int k = 0; k < nb; ++k) gJ_host[k] = h[k] + 0.25 * h[nb];
    return ED_OK;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

void terms_free(ed_basis *b)
{
    auto &t = b->terms;
    for (void *p : {t.words, (void *)t.off, (void *)t.cnt, (void *)t.xs, (void *)t.pair, (void *)t.cls, (void *)t.cls_chi,
                    (void *)t.next, (void *)t.adj})
        if (p) (void)hipFree(p);
    t.words = nullptr;
    t.off = nullptr;
    t.cnt = nullptr;
    t.xs = t.pair = t.cls = t.cls_chi = t.adj = nullptr;
    t.next = nullptr;
    b->device_bytes -= t.bytes;
    t.bytes = 0;
    t.couplings_ok = t.captured = false;
}

// One coefficient per orbit: couplings that differ in their last bits within an
// orbit (the check allows 1e-12) run the searching kernels, which read them
// bond by bond.  The classes get the first bond's then, for a captured H.v that
// reads stored terms when it is replayed.
bool terms_couplings_equal(const ed_basis *b, const double *J)
{
    std::vector<int> first(b->t.nb, -1);
    for (int k = 0; k < b->t.nb; ++k) {
        int &f = first[b->t.bond_orbit[k]];
        if (f < 0) f = k;
        if (J[k] != J[f]) return false;
    }
    return true;
}

// class coefficients of new couplings (ordered on the stream, which the
// caller synchronises before the host arrays here go: none do, they are
// copied first)
int terms_couplings(ed_basis *b, const double *J, const double *Jz, void *stream)
{
    auto &t = b->terms;
    if (!t.words) return ED_OK;
    hipStream_t st = (hipStream_t)stream;
    t.couplings_ok = false;
    const int W = b->dm.is_complex ? 4 : 2;
    std::vector<double> tab((size_t)t.n_cls * W, 0.0);
    const int n_chi = (int)t.chi_vals.size() / 2;
    for (int x = 0; x < n_chi; ++x)
        for (int o = 0; o < t.n_orb; ++o) {
            double *c = &tab[((size_t)x * t.n_orb + o) * W];
            const double jh = b->fermion ? -J[t.orbit_bond[o]] : 0.5 * J[t.orbit_bond[o]];
            c[0] = jh * t.chi_vals[2 * x];
            if (b->dm.is_complex) c[1] = jh * t.chi_vals[2 * x + 1];
            c[b->dm.is_complex ? 2 : 1] = b->fermion ? 0.0 : 0.5 * Jz[t.orbit_bond[o]];
        }
    HIP_TRY(hipMemcpyAsync(t.cls, tab.data(), tab.size() * 8, hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    t.couplings_ok = terms_couplings_equal(b, J) && terms_couplings_equal(b, Jz);
    return ED_OK;
}

template <typename AT, int NSC, bool FERMI>
static int fill_impl(ed_basis *b, const uint16_t *chi_class, const uint16_t *orbit, uint32_t pad, hipStream_t st)
{
    auto kern = k_terms_fill<AT, NSC, FERMI>;
    const int th = (int)b->dm.lds_total * 2 > lds_limit() ? 1024 : 512;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, th, b->dm.lds_total) != hipSuccess || per_cu < 1)
        per_cu = 1;
    // few slices: several waves share one, so that a short table is not one
    // wave's chain of searches
    const int64_t slices = b->terms.n_slices, waves = (int64_t)per_cu * num_cus() * (th / kWave);
    int parts = 1;
    while (parts < 16 && slices * parts * 2 <= waves) parts *= 2;
    const int64_t need = (slices * parts + th / kWave - 1) / (th / kWave);
    const int grid = (int)std::max<int64_t>(std::min<int64_t>((int64_t)per_cu * num_cus(), need), 1);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(th), b->dm.lds_total, st, b->dm, b->db, b->rep_index, (const uint64_t *)b->terms.off,
                       b->terms.stride, b->terms.cnt, (uint32_t *)b->terms.words, chi_class, orbit, b->terms.n_orb,
                       b->terms.ibits, pad, parts, slices);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(ED_ERR_HIP, "term search launch failed: %s", hipGetErrorString(e));
    return ED_OK;
}

// the search instances of the H.v kernels
template <typename AT, bool FERMI>
static int fill_ns(ed_basis *b, const uint16_t *cc, const uint16_t *orb, uint32_t pad, hipStream_t st)
{
    const int ns = b->dm.ns, nc = b->dm.n_chunks;
    if constexpr (FERMI) {
        if (ns == 4 && nc == 3) return fill_impl<AT, 35, true>(b, cc, orb, pad, st);
        if (ns == 4 && nc == 2) return fill_impl<AT, 34, true>(b, cc, orb, pad, st);
        return fill_impl<AT, 0, true>(b, cc, orb, pad, st);
    } else {
        constexpr int F = kStagedFlag;
        if (b->staged) {
            if (ns == 4 && nc == 1) return fill_impl<AT, 33 + F, false>(b, cc, orb, pad, st);
            if (ns == 4 && nc == 2) return fill_impl<AT, 34 + F, false>(b, cc, orb, pad, st);
            if (ns == 4 && nc == 3) return fill_impl<AT, 35 + F, false>(b, cc, orb, pad, st);
            if (ns == 2) return fill_impl<AT, 16 + F, false>(b, cc, orb, pad, st);
            if (ns == 3) return fill_impl<AT, 24 + F, false>(b, cc, orb, pad, st);
            if (ns == 4) return fill_impl<AT, 32 + F, false>(b, cc, orb, pad, st);
        }
        if (ns == 4 && nc == 1) return fill_impl<AT, 33, false>(b, cc, orb, pad, st);
        if (ns == 4 && nc == 2) return fill_impl<AT, 34, false>(b, cc, orb, pad, st);
        if (ns == 4 && nc == 3) return fill_impl<AT, 35, false>(b, cc, orb, pad, st);
        switch (ns) {
        case 2: return fill_impl<AT, 16, false>(b, cc, orb, pad, st);
        case 3: return fill_impl<AT, 24, false>(b, cc, orb, pad, st);
        case 4: return fill_impl<AT, 32, false>(b, cc, orb, pad, st);
        case 5: return fill_impl<AT, 40, false>(b, cc, orb, pad, st);
        case 6: return fill_impl<AT, 48, false>(b, cc, orb, pad, st);
        case 8: return fill_impl<AT, 64, false>(b, cc, orb, pad, st);
        case 9: return fill_impl<AT, 72, false>(b, cc, orb, pad, st);
        case 10: return fill_impl<AT, 80, false>(b, cc, orb, pad, st);
        default: return fill_impl<AT, 0, false>(b, cc, orb, pad, st);
        }
    }
}

// the rows, overwritten by the amplitudes of real sectors since the basis was
// built, for a search without the index
__global__ void k_slots_rows(const uint32_t *slot_of, char *slots, int slot_bytes, int64_t D)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < D; j += (int64_t)gridDim.x * blockDim.x)
        *(uint64_t *)(slots + (size_t)slot_of[j] * slot_bytes + 8) = (uint64_t)j;
}

static bool terms_possible(const ed_basis *b)
{
    return b->want_terms && b->db.index_mode == 0 && b->db.dim >= 1 && b->t.nb >= 1;
}

static size_t tuned_limit(const ed_basis *b)
{
    return b->tuning.stored_terms_mb > 0 ? (size_t)b->tuning.stored_terms_mb << 20 : SIZE_MAX;
}

// Most bytes of a table that a basis keeps: 1/16 of the device's memory, and at
// least half of it stays free, so that programs with many bases or large
// tensors have what they had without tables (small tables, up to 1/1024 of what
// is free, are kept in any case).
static size_t keep_limit(const ed_basis *b, size_t free_b, size_t total_b)
{
    const size_t half = total_b / 2;
    return std::min(tuned_limit(b), std::max(free_b / 1024, free_b > half ? std::min(total_b / 16, free_b - half) : (size_t)0));
}

// whether terms_build may find room, by half of the mean number of antiparallel
// bonds over all configurations (a sector's rows have more or less than that
// mean, by far less than a factor of two)
bool terms_wanted(const ed_basis *b)
{
    size_t free_b = 0, total_b = 0;
    if (!terms_possible(b)) return false;
    if (b->db.dim < (1 << 16)) return true;
    const double n = b->n_up, N = b->t.N, anti = 2.0 * n * (N - n) / (N * (N - 1.0));
    return hipMemGetInfo(&free_b, &total_b) == hipSuccess &&
           (double)b->db.dim * b->t.nb * 4.0 * 0.5 * anti <= (double)keep_limit(b, free_b, total_b);
}

// the first slices whose words take at most bytes; *groups: their groups.
// off is on the device: a binary search by single reads
static int64_t slices_that_fit(const uint64_t *off, int64_t slices, size_t bytes, uint64_t *groups, hipStream_t st)
{
    const uint64_t most = bytes / ((size_t)kWave * 16);
    int64_t lo = 0, hi = slices - 1;   // slices [0, lo) fit, their end is off[lo]
    *groups = 0;
    while (lo < hi) {
        const int64_t mid = hi - (hi - lo) / 2;
        uint64_t end = 0;
        if (hipMemcpyAsync(&end, off + mid, 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return 0;
        if (end <= most) {
            lo = mid;
            *groups = end;
        } else {
            hi = mid - 1;
        }
    }
    return lo;
}

void free_rep_index(ed_basis *b)
{
    if (b->rep_index.entries) (void)hipFree(b->rep_index.entries);
    if (b->rep_lists) (void)hipFree(b->rep_lists);
    b->rep_index = RepIndex{};
    b->rep_lists = nullptr;
}

// Builds the table, if the sector can have one: a hash-slot basis with bonds,
// a word that holds class and row, and a table within keep_limit.  Anything
// else leaves the basis without
// one, to the searching kernels; only an error of the device is returned.  A
// batched basis gives the classes of its elements (equal characters in every
// sector), whose coefficients are then the couplings alone.  A call's own
// table may take call_limit bytes; it holds the first slices where not all fit
// (an eighth at least, or none).
int terms_build(ed_basis *b, void *stream, const uint16_t *elem_class, int n_elem_class, size_t call_limit)
{
    hipStream_t st = (hipStream_t)stream;
    auto &t = b->terms;
    const int64_t D = b->db.dim;
    const int nb = b->t.nb, ng = b->t.ng;
    if (call_limit ? !terms_possible(b) : !terms_wanted(b)) return ED_OK;
    // distinct characters (fermions: and their negatives, for the sign)
    std::vector<uint16_t> cls((size_t)ng * 2);
    t.chi_vals.clear();
    for (int k = 0; elem_class && k < n_elem_class; ++k) {
        t.chi_vals.push_back(1.0);
        t.chi_vals.push_back(0.0);
    }
    if (elem_class) std::copy(elem_class, elem_class + ng, cls.begin());
    for (int sgn = 0; !elem_class && sgn < (b->fermion ? 2 : 1); ++sgn)
        for (int g = 0; g < ng; ++g) {
            const double re = sgn ? -b->chi_host[2 * g] : b->chi_host[2 * g];
            const double im = b->dm.is_complex ? (sgn ? -b->chi_host[2 * g + 1] : b->chi_host[2 * g + 1]) : 0.0;
            size_t k = 0;
            while (k < t.chi_vals.size() && !(t.chi_vals[k] == re && t.chi_vals[k + 1] == im)) k += 2;
            if (k / 2 >= (size_t)kMaxClasses) return ED_OK;
            if (k == t.chi_vals.size()) {
                t.chi_vals.push_back(re);
                t.chi_vals.push_back(im);
            }
            cls[(size_t)sgn * ng + g] = (uint16_t)(k / 2);
        }
    std::vector<uint16_t> orb(nb);
    t.orbit_bond.clear();
    for (int k = 0; k < nb; ++k) {
        orb[k] = (uint16_t)b->t.bond_orbit[k];
        if ((size_t)orb[k] >= t.orbit_bond.size()) t.orbit_bond.resize(orb[k] + 1, -1);
        if (t.orbit_bond[orb[k]] < 0) t.orbit_bond[orb[k]] = k;
    }
    t.n_orb = (int)t.orbit_bond.size();
    t.n_cls = (int)(t.chi_vals.size() / 2) * t.n_orb + 1;   // and the padding
    if (t.n_cls > kMaxClasses) return ED_OK;
    int cbits = 1;
    while ((1 << cbits) < t.n_cls) ++cbits;
    t.ibits = 32 - cbits;
    const size_t vec = ((size_t)D + 1) * (b->dm.is_complex ? 16 : 8);
    if ((uint64_t)D >= (1ull << t.ibits) || vec > 0xFFFFFFFFull) return ED_OK;

    const int64_t slices = (D + kWave - 1) / kWave;
    auto give_up = [&]() {
        (void)hipGetLastError();
        terms_free(b);
        return ED_OK;
    };
    auto take = [&](void **p, size_t bytes) {
        if (hipMalloc(p, bytes) != hipSuccess) {
            *p = nullptr;
            return false;
        }
        t.bytes += (int64_t)bytes;
        b->device_bytes += (int64_t)bytes;
        return true;
    };
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) return give_up();
    if (!take((void **)&t.cnt, (size_t)slices * 4)) return give_up();
    // small sectors take the longest possible slices at a fixed stride; others
    // are counted first
    constexpr size_t kGroupBytes = (size_t)kWave * 16;
    uint64_t groups = (uint64_t)slices * (uint64_t)((nb + 3) / 4);
    if (groups * kGroupBytes <= (16u << 20)) {
        t.stride = (uint32_t)((nb + 3) / 4);
    } else {
        t.stride = 0;
        const unsigned g = (unsigned)std::min<int64_t>((slices + 3) / 4, (int64_t)num_cus() * 32);
        hipLaunchKernelGGL(k_terms_count, dim3(g), dim3(256), 0, st, b->dm, b->db.states, D, t.cnt);
        HIP_TRY(hipGetLastError());
        if (!take((void **)&t.off, (size_t)slices * 8)) return give_up();
        int rc = scan_counts(t.cnt, t.off, (uint64_t)slices, st);
        if (rc == ED_ERR_OOM) return give_up();
        if (rc) return rc;
        uint64_t last_off = 0;
        uint32_t last_cnt = 0;
        HIP_TRY(hipMemcpyAsync(&last_off, t.off + slices - 1, 8, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipMemcpyAsync(&last_cnt, t.cnt + slices - 1, 4, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        groups = last_off + last_cnt;
    }
    const size_t limit = call_limit ? std::min(call_limit, tuned_limit(b)) : keep_limit(b, free_b, total_b);
    t.n_slices = slices;
    if (groups * kGroupBytes + vec > limit) {
        if (!call_limit || t.stride || limit < vec) return give_up();
        t.n_slices = slices_that_fit(t.off, slices, limit - vec, &groups, st);
        if (t.n_slices < std::max<int64_t>(slices / 8, 1)) return give_up();
    }
    const size_t bytes = std::max<size_t>(groups, 1) * kGroupBytes;
    // the scaled input exceeds the L2s: slices from a counter
    const bool counted = lz_per_slice(b) && !elem_class;
    const size_t clsb = (size_t)t.n_cls * (b->dm.is_complex ? 32 : 16);
    void *d_cls = nullptr;   // chi classes and bond orbits, needed by the search only
    if (!take(&t.words, bytes) || (!elem_class && !take((void **)&t.xs, vec)) || !take((void **)&t.cls, clsb) ||
        !take((void **)&t.cls_chi, clsb / 2) ||
        (counted && !take((void **)&t.next, 8 * kNextStride * 4)) ||
        hipMalloc(&d_cls, (cls.size() + orb.size()) * 2) != hipSuccess)
        return give_up();
    std::vector<double> chi((size_t)t.n_cls * (b->dm.is_complex ? 2 : 1), 0.0);
    for (int k = 0; k + 1 < t.n_cls; ++k) {
        const double *v = &t.chi_vals[2 * (k / t.n_orb)];
        if (b->dm.is_complex) {
            chi[2 * k] = v[0];
            chi[2 * k + 1] = v[1];
        } else {
            chi[k] = v[0];
        }
    }
    cls.insert(cls.end(), orb.begin(), orb.end());
    hipError_t e = hipMemcpyAsync(d_cls, cls.data(), cls.size() * 2, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(t.cls_chi, chi.data(), chi.size() * 8, hipMemcpyHostToDevice, st);
    if (e == hipSuccess && t.xs)
        e = hipMemsetAsync((char *)t.xs + vec - (b->dm.is_complex ? 16 : 8), 0, b->dm.is_complex ? 16 : 8, st);
    if (e == hipSuccess && call_limit) {
        hipLaunchKernelGGL(k_slots_rows, dim3((unsigned)std::min<int64_t>((D + 255) / 256, 1 << 20)), dim3(256), 0, st,
                           b->db.slot_of, b->db.slots, b->dm.is_complex ? 32 : 16, D);
        e = hipGetLastError();
    }
    int rc = ED_OK;
    if (e == hipSuccess) {
        const uint32_t pad = (uint32_t)(t.n_cls - 1) << t.ibits | (uint32_t)D;
        const uint16_t *cc = (const uint16_t *)d_cls, *ob = cc + 2 * (size_t)ng;
        if (b->fermion)
            rc = b->dm.act_bytes == 2 ? fill_ns<FermiU16, true>(b, cc, ob, pad, st) : fill_ns<uint32_t, true>(b, cc, ob, pad, st);
        else
            rc = b->dm.act_bytes == 1   ? fill_ns<uint8_t, false>(b, cc, ob, pad, st)
                 : b->dm.act_bytes == 2 ? fill_ns<uint16_t, false>(b, cc, ob, pad, st)
                                        : fill_ns<uint32_t, false>(b, cc, ob, pad, st);
        const hipError_t es = hipStreamSynchronize(st);
        if (e == hipSuccess) e = es;
    }
    (void)hipFree(d_cls);
    if (rc) return rc;
    if (e != hipSuccess) return set_error(ED_ERR_HIP, "term search failed: %s", hipGetErrorString(e));
    b->J_cache.clear();
    return ED_OK;
}

}  // namespace ed

extern "C" int64_t ed_basis_terms_bytes(const ed_basis_t *b) { return b && b->terms.words ? b->terms.bytes : 0; }

extern "C" int ed_basis_release_terms(ed_basis_t *b)
{
    if (!b) return ed::set_error(ED_ERR_ARG, "null basis");
    b->want_terms = false;
    if (!b->terms.words) return ED_OK;
    if (hipDeviceSynchronize() != hipSuccess) return ed::set_error(ED_ERR_HIP, "device synchronisation");
    ed::terms_free(b);
    return ED_OK;
}
