// analyse.cpp -- descriptor analyser: the host-side stand-in for the paper's
// code generator (Sec. 3.2-3.3, Sec. 6).  Runs once per contraction shape and
// makes no HIP call.
//
//   1. parse and validate the three mode lists (Sec. 2.2, footnote 9);
//   2. classify indices into I_m, I_n, I_k (Listing 5: I_m = A ∩ C,
//      I_n = B ∩ C, I_k = A ∩ B);
//   3. drop extent-1 indices and merge indices of one set that are adjacent
//      in memory in every tensor holding them into super-indices (Sec. 6,
//      footnote 18, applied to strides so that it also covers non-dense
//      views);
//   4. choose the row and column operands of the macro-kernel: C's
//      stride-one index goes to the column side, where the kernel stores C
//      contiguously (the operand exchange of Listing 7, mirrored for the
//      MFMA result layout);
//   5. order every set so each operand's stride-one index leads where
//      possible (Sec. 3.2.1: keep the stride-one index inside the packed
//      sub-tensor);
//   6. choose the tile shape and the K box -- a sub-tensor of fixed shape
//      over the contracted indices, splitting one index into blocks
//      (Sec. 3.2.1, Examples 1-2: index reinterpretation) -- and the gather
//      mode of each operand.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <limits>
#include <cctype>
#include <new>
#include <sstream>

#include "plan.hpp"
#include "tiles.hpp"

namespace gett {
namespace {

gett_status_t parse_modes(const char *s, std::vector<std::string> &out)
{
    out.clear();
    if (!s) return GETT_ERROR_INVALID_VALUE;
    if (!strchr(s, ',')) {
        for (const char *p = s; *p; ++p)
            if (*p != ' ') out.push_back(std::string(1, *p));
        return GETT_SUCCESS;
    }
    std::string cur;
    for (const char *p = s;; ++p) {
        if (*p == ',' || *p == 0) {
            if (cur.empty()) {
                if (*p == 0 && !out.empty()) break;   // one trailing comma
                return GETT_ERROR_INVALID_INDICES;
            }
            out.push_back(cur);
            cur.clear();
            if (*p == 0) break;
        } else if (*p != ' ') {
            cur.push_back(*p);
        }
    }
    return GETT_SUCCESS;
}

struct Tensor {
    std::vector<std::string> modes;
    std::vector<int64_t> ext, str;
    int find(const std::string &n) const
    {
        for (size_t i = 0; i < modes.size(); ++i)
            if (modes[i] == n) return (int)i;
        return -1;
    }
};

gett_status_t load_tensor(const char *m, const int64_t *e, const int64_t *s, Tensor &t)
{
    gett_status_t st = parse_modes(m, t.modes);
    if (st != GETT_SUCCESS) return st;
    const size_t n = t.modes.size();
    if (n > GETT_MAX_RANK) return GETT_ERROR_NOT_SUPPORTED;
    if (n && !e) return GETT_ERROR_INVALID_VALUE;
    for (size_t i = 0; i < n; ++i)
        for (size_t j = i + 1; j < n; ++j)
            if (t.modes[i] == t.modes[j]) return GETT_ERROR_INVALID_INDICES;
    t.ext.assign(e, e + n);
    for (int64_t v : t.ext)
        if (v < 0 || v > INT32_MAX) return GETT_ERROR_INVALID_VALUE;
    if (s) {
        t.str.assign(s, s + n);
    } else {   // Fortran layout: the first index is stride-one (Sec. 2.2)
        t.str.resize(n);
        int64_t acc = 1;
        for (size_t i = 0; i < n; ++i) {
            t.str[i] = acc;
            acc *= std::max<int64_t>(t.ext[i], 1);
        }
    }
    for (size_t i = 0; i < n; ++i) {
        if (t.str[i] < 0) return GETT_ERROR_INVALID_VALUE;
        if (t.ext[i] > 1 && t.str[i] < 1) return GETT_ERROR_INVALID_VALUE;
    }
    return GETT_SUCCESS;
}

// Largest element offset of a tensor (INT64_MAX beyond 2^62).
int64_t max_offset(const Tensor &t)
{
    const int64_t cap = (int64_t)1 << 62;
    int64_t m = 0;
    for (size_t i = 0; i < t.modes.size(); ++i) {
        if (t.ext[i] <= 1) continue;
        if (t.str[i] >= cap || (t.ext[i] - 1) > cap / t.str[i]) return INT64_MAX;
        m += (t.ext[i] - 1) * t.str[i];
        if (m >= cap) return INT64_MAX;
    }
    return m;
}

}  // namespace

// Strides that may send two elements to one address are refused: sorted by
// stride, each index must step over the whole span of the previous ones.
bool strides_injective(int n, const int64_t *ext, const int64_t *str)
{
    std::vector<std::pair<int64_t, int64_t>> v;   // (stride, extent)
    for (int i = 0; i < n; ++i)
        if (ext[i] > 1) v.push_back({str[i], ext[i]});
    std::sort(v.begin(), v.end());
    int64_t span = 1;   // one past the largest offset reachable so far
    for (auto &p : v) {
        if (p.first < span) return false;
        span = p.first * (p.second - 1) + span;
    }
    return true;
}

namespace {

bool c_is_injective(const Tensor &c)
{
    return strides_injective((int)c.modes.size(), c.ext.data(), c.str.data());
}

// Merge p then q (p fastest) when q follows p in memory in every tensor that
// holds them (Sec. 6, footnote 18).
void merge_set(std::vector<Index> &set, bool useA, bool useB, bool useC,
               std::vector<std::string> &log)
{
    bool changed = true;
    while (changed) {
        changed = false;
        for (size_t p = 0; p < set.size() && !changed; ++p)
            for (size_t q = 0; q < set.size() && !changed; ++q) {
                if (p == q) continue;
                const Index &P = set[p], &Q = set[q];
                auto follows = [&](int64_t sp, int64_t sq) { return sq == sp * P.extent; };
                if (useA && !follows(P.strA, Q.strA)) continue;
                if (useB && !follows(P.strB, Q.strB)) continue;
                if (useC && !follows(P.strC, Q.strC)) continue;
                Index M = P;
                M.name = "(" + P.name + "," + Q.name + ")";
                M.extent = P.extent * Q.extent;
                log.push_back(M.name);
                set[p] = M;
                set.erase(set.begin() + q);
                changed = true;
            }
    }
}

const TileShape &tile_shape(gett_dtype_t dt, int t)
{
    return dt == GETT_FLOAT32 ? kTilesF32[t] : kTilesF64[t];
}
int num_tiles(gett_dtype_t dt) { return dt == GETT_FLOAT32 ? kNumTilesF32 : kNumTilesF64; }

void json_set(std::ostringstream &o, const char *key, const std::vector<Index> &set, bool A, bool B,
              bool C)
{
    o << "\"" << key << "\":[";
    for (size_t i = 0; i < set.size(); ++i) {
        const Index &x = set[i];
        o << (i ? "," : "") << "{\"name\":\"" << x.name << "\",\"extent\":" << x.extent;
        if (A) o << ",\"strideA\":" << x.strA;
        if (B) o << ",\"strideB\":" << x.strB;
        if (C) o << ",\"strideC\":" << x.strC;
        o << "}";
    }
    o << "]";
}

}  // namespace

Hooks read_hooks()
{
    Hooks h;
    const struct {
        const char *name;
        const char **slot;
    } vars[] = {{"GETT_FORCE_TILE", &h.forceTile},     {"GETT_FORCE_KIND", &h.forceKind},
                {"GETT_FORCE_KSLICES", &h.forceKslices}, {"GETT_SPLIT_F", &h.splitF},
                {"GETT_C_ORDER", &h.cOrder},           {"GETT_XCD_REMAP", &h.xcdRemap},
                {"GETT_LANE_PERM", &h.lanePerm},       {"GETT_TAIL_WGS", &h.tailWgs}};
    for (const auto &v : vars) {
        *v.slot = getenv(v.name);
        if (*v.slot) h.text += std::string(v.name) + "=" + *v.slot + ";";
    }
    // the text goes into gett_plan_describe's JSON: keep it to plain characters
    for (char &c : h.text)
        if (!(isalnum((unsigned char)c) || c == '_' || c == '=' || c == ';' || c == '-' ||
              c == '.'))
            c = '?';
    return h;
}

const char *kind_name(int k)
{
    return k == 1   ? "stream"
           : k == 2 ? "kslices"
           : k == 3 ? "tail"
           : k == 4 ? "direct"
           : k == 5 ? "direct-stream"
           : k == 6 ? "direct-element"
                    : "macro";
}

// Workgroups of a tile resident on one CU at once: the wavefronts per SIMD its
// register budget allows (a workgroup of four wavefronts puts one on each
// SIMD), within the 160 KB of LDS its packed panels take.
static double tail_occupancy(const TileShape &c, double itemB)
{
    const double lds = (double)c.nbuf * c.kt * (c.mt + c.nt + 8) * itemB;
    return std::max(1.0, std::min((double)c.wpe, std::floor(160.0 * 1024.0 / lds)));
}

// Time one CU takes, in units of one K box on a SIMD shared by two or more
// wavefronts, to run `full` workgroups of `nb` boxes and then `tail`
// workgroups of `len` boxes, `occ` of them resident at once (in that order:
// the dispatcher deals workgroups in order of their index).  The resident
// workgroups share the SIMDs evenly; a wavefront left alone on its SIMD runs
// at 0.64 of the rate of two (measured on MI355X: it waits for its own
// gathers and LDS reads).
static double cu_time(int occ, int full, double nb, int tail, double len)
{
    // equal runs finish together: whole rounds, and a last one at the rate of
    // what is left of it
    if (tail == 0) {
        const bool lone = occ >= 2 && full % std::min(occ, 8) == 1;
        return nb * (lone ? full - 1 + 1.0 / 0.64 : full);
    }
    // (at most eight wavefronts per SIMD, so at most eight workgroups here)
    double left[8];
    int held = 0, next = 0;
    occ = std::min(occ, 8);
    const int n = full + tail;
    auto work = [&](int i) { return i < full ? nb : len; };
    while (next < n && held < occ) left[held++] = work(next++);
    double t = 0.0;
    while (held > 0) {
        // (a tile that holds one wavefront per SIMD anyway has that rate in
        // its measured efficiency)
        const double rate = (held >= 2 || occ < 2 ? 1.0 : 0.64) / (double)held;   // per unit, each
        const double step = *std::min_element(left, left + held);
        t += step / rate;
        int still = 0;
        for (int i = 0; i < held; ++i)
            if (left[i] - step > 1e-9) left[still++] = left[i] - step;
        held = still;
        while (next < n && held < occ) left[held++] = work(next++);
    }
    return t;
}

// Stream-K tail shape for T tiles of nb boxes over G tail workgroups:
// whole tiles for the complete rounds of G, the boxes of the rest in equal
// runs; every tail workgroup gets boxes.
struct TailShape {
    int64_t full = 0, wgs = 0, len = 0;
};
// Chain behind an element of a tile of nb boxes that are dealt in runs of len,
// as a share of the nb: the pieces' squares over nb squared, averaged over where
// the runs' ends fall (a sum's squared error grows with the square of each
// piece's length over the whole's).
static double tail_chain(int64_t len, int64_t nb)
{
    const double l = (double)len, n = (double)nb;
    if (nb % len == 0 || len % nb == 0) return std::min(1.0, l / n);
    return l < n ? l / n * (1.0 - l / (3.0 * n)) : 1.0 - n / (3.0 * l);
}
static TailShape tail_shape(int64_t T, int64_t nb, int64_t G)
{
    TailShape s;
    int64_t rem = T % G;
    if (rem == 0) rem = std::min<int64_t>(G, T);
    const int64_t boxes = rem * nb;
    s.len = (boxes + std::min(G, boxes) - 1) / std::min(G, boxes);
    s.full = T - rem;
    s.wgs = (boxes + s.len - 1) / s.len;
    return s;
}

namespace {

const char *mode_name(int m)
{
    return m == kGatherRowVec         ? "row-vector"
           : m == kGatherKVec         ? "k-vector"
           : m == kGatherRowVecStrided ? "row-vector-strided"
           : m == kGatherKVecStrided  ? "k-vector-strided"
                                      : "scalar";
}

}  // namespace

gett_status_t front_end(Analysis &an, gett_dtype_t dtype, const char *mC, const int64_t *eC,
                        const int64_t *sC, const char *mA, const int64_t *eA, const int64_t *sA,
                        const char *mB, const int64_t *eB, const int64_t *sB, int rank[3],
                        bool offsets31)
{
    if (dtype != GETT_FLOAT32 && dtype != GETT_FLOAT64) return GETT_ERROR_INVALID_VALUE;
    Tensor A, B, C;
    gett_status_t st;
    if ((st = load_tensor(mC, eC, sC, C)) != GETT_SUCCESS) return st;
    if ((st = load_tensor(mA, eA, sA, A)) != GETT_SUCCESS) return st;
    if ((st = load_tensor(mB, eB, sB, B)) != GETT_SUCCESS) return st;
    rank[0] = (int)C.modes.size();
    rank[1] = (int)A.modes.size();
    rank[2] = (int)B.modes.size();

    // ---- classification (Sec. 2.2; Listing 5: the three intersections) ----
    for (size_t i = 0; i < C.modes.size(); ++i) {
        const int ia = A.find(C.modes[i]), ib = B.find(C.modes[i]);
        if ((ia >= 0) == (ib >= 0)) return GETT_ERROR_INVALID_INDICES;   // in both or neither
        Index x;
        x.name = C.modes[i];
        x.extent = C.ext[i];
        x.strC = C.str[i];
        if (ia >= 0) {
            if (A.ext[ia] != C.ext[i]) return GETT_ERROR_INVALID_INDICES;
            x.strA = A.str[ia];
            an.Im.push_back(x);
        } else {
            if (B.ext[ib] != C.ext[i]) return GETT_ERROR_INVALID_INDICES;
            x.strB = B.str[ib];
            an.In.push_back(x);
        }
    }
    for (size_t i = 0; i < A.modes.size(); ++i) {
        if (C.find(A.modes[i]) >= 0) continue;
        const int ib = B.find(A.modes[i]);
        if (ib < 0) return GETT_ERROR_INVALID_INDICES;
        if (B.ext[ib] != A.ext[i]) return GETT_ERROR_INVALID_INDICES;
        Index x;
        x.name = A.modes[i];
        x.extent = A.ext[i];
        x.strA = A.str[i];
        x.strB = B.str[ib];
        an.Ik.push_back(x);
    }
    for (size_t i = 0; i < B.modes.size(); ++i)
        if (C.find(B.modes[i]) < 0 && A.find(B.modes[i]) < 0) return GETT_ERROR_INVALID_INDICES;

    an.maxOffA = max_offset(A);
    an.maxOffB = max_offset(B);
    an.maxOffC = max_offset(C);
    const int64_t lim = offsets31 ? (int64_t)INT32_MAX : INT64_MAX;
    if (an.maxOffA >= lim || an.maxOffB >= lim || an.maxOffC >= lim) return GETT_ERROR_NOT_SUPPORTED;
    if (!c_is_injective(C)) return GETT_ERROR_NOT_SUPPORTED;

    for (auto &x : an.Im) { an.sizeM *= x.extent; }
    for (auto &x : an.In) { an.sizeN *= x.extent; }
    for (auto &x : an.Ik) { an.sizeK *= x.extent; }
    an.emptyC = an.sizeM == 0 || an.sizeN == 0;
    an.emptySum = an.sizeK == 0;

    // ---- drop extent-1 indices, merge (footnote 18) ----
    auto drop1 = [](std::vector<Index> &s) {
        s.erase(std::remove_if(s.begin(), s.end(), [](const Index &x) { return x.extent == 1; }),
                s.end());
    };
    drop1(an.Im);
    drop1(an.In);
    drop1(an.Ik);
    if (!an.emptyC && !an.emptySum) {
        merge_set(an.Im, true, false, true, an.merges);
        merge_set(an.In, false, true, true, an.merges);
        merge_set(an.Ik, true, true, false, an.merges);
    }

    return GETT_SUCCESS;
}

gett_status_t analyse(gett_plan_s &plan, gett_dtype_t dtype, const char *mC, const int64_t *eC,
                      const int64_t *sC, const char *mA, const int64_t *eA, const int64_t *sA,
                      const char *mB, const int64_t *eB, const int64_t *sB, uint32_t flags,
                      const Choice *force)
{
    Analysis an;
    int rank[3];
    const gett_status_t st =
        front_end(an, dtype, mC, eC, sC, mA, eA, sA, mB, eB, sB, rank, false);
    if (st != GETT_SUCCESS) return st;

    // ---- operand roles: C's stride-one index on the column (y) side ----
    bool swap = false;
    {
        int64_t best = INT64_MAX;
        int where = 0;   // 1: I_m, 2: I_n
        for (auto &x : an.Im)
            if (x.strC < best) { best = x.strC; where = 1; }
        for (auto &x : an.In)
            if (x.strC < best) { best = x.strC; where = 2; }
        swap = where == 1 && !(flags & GETT_FLAG_NO_SWAP);
    }
    an.swapped = swap;
    std::vector<Index> Ix = swap ? an.In : an.Im;
    std::vector<Index> Iy = swap ? an.Im : an.In;
    std::vector<Index> Ik = an.Ik;
    auto sX = [swap](const Index &x) { return swap ? x.strB : x.strA; };
    auto sY = [swap](const Index &x) { return swap ? x.strA : x.strB; };

    // ---- loop orders (stride-one index first where it helps) ----
    std::stable_sort(Iy.begin(), Iy.end(), [](const Index &a, const Index &b) { return a.strC < b.strC; });
    std::stable_sort(Ix.begin(), Ix.end(), [&](const Index &a, const Index &b) { return sX(a) < sX(b); });
    {
        int64_t minX = INT64_MAX, minY = INT64_MAX;
        bool xInK = false, yInK = false;
        for (auto &x : Ix) if (sX(x) < minX) { minX = sX(x); xInK = false; }
        for (auto &x : Ik) if (sX(x) < minX) { minX = sX(x); xInK = true; }
        for (auto &x : Iy) if (sY(x) < minY) { minY = sY(x); yInK = false; }
        for (auto &x : Ik) if (sY(x) < minY) { minY = sY(x); yInK = true; }
        const bool byY = !xInK && yInK;
        std::stable_sort(Ik.begin(), Ik.end(), [&](const Index &a, const Index &b) {
            return byY ? sY(a) < sY(b) : sX(a) < sX(b);
        });
    }
    // An empty set acts as one index of extent 1 (Sec. 2.2 assumes non-empty sets).
    auto virt = [](std::vector<Index> &s) {
        if (s.empty()) {
            Index v;
            v.name = "1";
            s.push_back(v);
        }
    };
    virt(Ix);
    virt(Iy);
    virt(Ik);
    if ((int)Ix.size() > kMaxDims || (int)Iy.size() > kMaxDims || (int)Ik.size() > kMaxDims)
        return GETT_ERROR_NOT_SUPPORTED;

    // ---- K box for a given box depth: whole leading contracted indices,
    //      then a block of one index (index reinterpretation) ----
    const int VW = dtype == GETT_FLOAT32 ? 4 : 2;
    const int64_t sizeX = swap ? an.sizeN : an.sizeM;
    const int64_t sizeY = swap ? an.sizeM : an.sizeN;
    int nk = (int)Ik.size();
    // A contracted stride-one run gathered as vectors needs whole vectors per block.
    auto kvec_ok = [&](auto strOf) {
        if (strOf(Ik[0]) != 1) return false;
        if (Ik[0].extent % VW) return false;
        for (size_t i = 1; i < Ik.size(); ++i)
            if (strOf(Ik[i]) % VW) return false;
        return true;
    };
    const bool wantKvec = !(flags & GETT_FLAG_SCALAR) && (kvec_ok(sX) || kvec_ok(sY));
    int kvecIdx = 0;   // contracted index that vector gathers run along (1 after a K split)
    struct Box {
        int kj;
        int64_t tj, kbox, nblk, nsteps;
    };
    // K box of depth kt over the contracted set K (in walk order); kvi is the
    // index that contracted vector gathers run along.
    auto box_on = [&](const std::vector<Index> &K, int kvi, int kt) {
        const int nK = (int)K.size();
        Box b;
        b.kj = 0;
        int64_t prefix = 1;
        while (b.kj < nK - 1 && prefix * K[b.kj].extent <= kt) {
            prefix *= K[b.kj].extent;
            ++b.kj;
        }
        int64_t tj = std::max<int64_t>(1, std::min<int64_t>(K[b.kj].extent, kt / prefix));
        // The block of the index that vectors run along holds whole vectors.
        // A block length that divides the index (no ragged last block) is
        // preferred unless that would lose more than half of the box (92 in
        // blocks of 4 would be 23 boxes an eighth full, against 32, 32, 28).
        const bool vec = b.kj == kvi && (wantKvec || kvi > 0);
        const int64_t step = vec ? VW : 1;
        const int64_t top = vec && tj >= VW ? (tj / VW) * VW : tj;
        if (top >= step) {
            int64_t best = top;
            for (int64_t t = top; t >= step; t -= step)
                if (K[b.kj].extent % t == 0) { best = t; break; }
            tj = best * 2 > top ? best : top;
        }
        b.tj = tj;
        b.kbox = prefix * tj;
        b.nblk = (K[b.kj].extent + tj - 1) / tj;
        b.nsteps = b.nblk;
        for (int i = b.kj + 1; i < nK; ++i) b.nsteps *= K[i].extent;
        if (an.emptySum) b.nsteps = 0;
        return b;
    };
    auto box_for = [&](int kt) { return box_on(Ik, kvecIdx, kt); };

    // ---- index splitting helpers (used by the model and by the plan; see
    //      the splitting step below) ----
    auto split_front = [](std::vector<Index> &set, size_t u, size_t v, int64_t f) {
        Index in = set[u], out = set[u];
        in.extent = f;
        in.name = set[u].name + "<" + std::to_string(f);
        out.extent = set[u].extent / f;
        out.name = set[u].name + ">" + std::to_string(f);
        out.strA *= f;
        out.strB *= f;
        out.strC *= f;
        std::vector<Index> next;
        next.push_back(in);
        next.push_back(set[v]);
        if (out.extent > 1) next.push_back(out);
        for (size_t i = 0; i < set.size(); ++i)
            if (i != u && i != v) next.push_back(set[i]);
        set.swap(next);
    };
    auto pow2_part = [](int64_t e) { return e & -e; };
    auto unit_in = [](const std::vector<Index> &set, auto strOf) -> int {
        for (size_t i = 0; i < set.size(); ++i)
            if (strOf(set[i]) == 1 && set[i].extent > 1) return (int)i;
        return -1;
    };
    auto aligned = [&](const std::vector<Index> &set, auto strOf, int skip) {
        for (size_t i = 0; i < set.size(); ++i)
            if ((int)i != skip && strOf(set[i]) % VW) return false;
        return true;
    };
    const bool maySplit = !(flags & (GETT_FLAG_SCALAR | GETT_FLAG_NO_SPLIT)) && !an.emptyC &&
                          !an.emptySum;
    const int splitXK = unit_in(Ik, sX), splitYK = unit_in(Ik, sY);
    // K-box split for a box of depth kt: X's stride-one contracted index u
    // blocked by f in front of Y's stride-one contracted index v.  X runs of f
    // (a multiple of VW), at least two vectors of v per box line when the
    // box allows.  Returns f (0: no split) and the split set in `trial`.
    auto k_split = [&](int kt, std::vector<Index> &trial) -> int64_t {
        if (!maySplit || splitXK < 0 || splitYK < 0 || splitXK == splitYK ||
            Ik[splitYK].extent % VW || (int)Ik.size() >= kMaxDims)
            return 0;
        int64_t cap = 1;
        while (cap * 2 * VW <= kt) cap *= 2;
        int64_t f = std::min<int64_t>(pow2_part(Ik[splitXK].extent), cap);
        while (f > VW && f * VW * 2 > kt) f /= 2;
        trial = Ik;
        split_front(trial, (size_t)splitXK, (size_t)splitYK, f);
        if (f >= VW && kt % (f * VW) == 0 && aligned(trial, sY, 1) && aligned(Iy, sY, -1)) return f;
        return 0;
    };

    // Order of the boxes of a direct-load kernel after a K split, Ik = (u_in,
    // v, u_out, ...): a box is u_in (f positions of X's stride-one index) by
    // kt / f positions of v (Y's), so it uses f elements of each of X's cache
    // lines and kt / f of Y's.  Walking all of v first returned to X's lines
    // only after every block of v, from HBM by then: the rest of a line was
    // fetched again for each box.  Here the boxes that share X's lines come
    // first, then those that share Y's: (u_in, v_in, u_mid, v_mid, u_out,
    // v_out, ...), u_mid and v_mid the boxes per 128-byte line.  v has to
    // divide into whole blocks (else the order stays).  Measured on the
    // 7056 x 8064 x 9216 fp32 contraction: 10.19 ms, in this order 9.53 ms.
    // The macro-kernels keep the plain order, which measured 2-10% faster on
    // their shallower boxes and K slices.
    auto walk_lines = [&](int kt) {
        const int64_t line = dtype == GETT_FLOAT32 ? 32 : 16;   // elements of 128 bytes
        const int64_t f = Ik[0].extent, vin = kt / f;
        if ((int)Ik.size() + 3 > kMaxDims || Ik[1].extent % vin) return;
        auto part = [](const Index &x, int64_t skip, int64_t ext, const char *tag, int64_t n) {
            Index p = x;
            p.extent = ext;
            p.name = x.name + tag + std::to_string(n);
            p.strA *= skip;
            p.strB *= skip;
            p.strC *= skip;
            return p;
        };
        auto divisor = [](int64_t n, int64_t cap) {
            int64_t d = std::max<int64_t>(1, std::min(n, cap));
            while (n % d) --d;
            return d;
        };
        const Index v = Ik[1];
        // u_out, where the split left one, has the name of no other index
        const bool hasU = Ik.size() > 2 && Ik[2].strA == Ik[0].strA * f && Ik[2].strB == Ik[0].strB * f;
        std::vector<Index> next = {Ik[0], part(v, 1, vin, "<", vin)};
        const int64_t rv = v.extent / vin, n = divisor(rv, line / vin);
        const int64_t m = hasU ? divisor(Ik[2].extent, line / f) : 1;
        if (m > 1) next.push_back(part(Ik[2], 1, m, "|", m));
        if (n > 1) next.push_back(part(v, vin, n, "|", n));
        if (hasU && Ik[2].extent > m) next.push_back(part(Ik[2], m, Ik[2].extent / m, "|>", m));
        if (rv > n) next.push_back(part(v, vin * n, rv / n, ">", vin * n));
        for (size_t i = hasU ? 3 : 2; i < Ik.size(); ++i) next.push_back(Ik[i]);
        Ik.swap(next);
        nk = (int)Ik.size();
    };

    // ---- tile shape: the paper ranks candidates with a performance model
    //      (Sec. 3.4: macro-kernel time from flops / (peak * penalty), packing
    //      and unpacking time from bytes / bandwidth).  Here: MFMA time of the
    //      busiest SIMD (the tiles' wavefronts are dealt to the 1024 SIMDs of
    //      256 CUs; each wavefront's share of a tile, padding included, runs
    //      at the sustained fraction of one SIMD's peak) against the C stream
    //      through HBM at the bandwidth the tile sustains; the longer one
    //      bounds the time. ----
    const double itemB = dtype == GETT_FLOAT32 ? 4.0 : 8.0;
    const double peakSimd = (dtype == GETT_FLOAT32 ? 157.3e12 : 78.6e12) / 1024.0;
    const double bytesX = itemB * (double)sizeX * (double)an.sizeK;
    const double bytesY = itemB * (double)sizeY * (double)an.sizeK;
    const double bytesC = itemB * (double)sizeX * (double)sizeY;
    // When the row and column operands are stride-one along different
    // contracted indices, the K box is split between them (below) and both
    // are gathered in short runs whose cache lines are reused only many
    // boxes later; without a second LDS buffer the gather latency of every
    // box is exposed (measured on MI355X: 1.4-1.8x slower than the
    // double-buffered tiles of the same depth).
    // Each tile's K box is priced on the contracted order that tile gets.
    const Hooks hk = read_hooks();
    const char *ft = hk.forceTile;
    const char *fk = hk.forceKind;
    // An operand gathers in vectors when its stride-one index leads its free
    // order or the contracted order (before any index split).
    auto vecable = [&](const std::vector<Index> &I, auto strOf) {
        return strOf(I[0]) == 1 || strOf(Ik[0]) == 1;
    };
    const bool slowGather = (flags & GETT_FLAG_SCALAR) || !vecable(Ix, sX) || !vecable(Iy, sY);
    // Whether the operand's extents and strides let it gather in 16-byte
    // vectors, in the orders as they stand (no split, no C order).
    auto vectors = [&](const std::vector<Index> &I, auto strOf) {
        const bool row = strOf(I[0]) == 1 && I[0].extent % VW == 0 && aligned(I, strOf, 0) &&
                         aligned(Ik, strOf, -1);
        return !(flags & GETT_FLAG_SCALAR) && (row || (kvec_ok(strOf) && aligned(I, strOf, -1)));
    };
    const bool vecX = vectors(Ix, sX), vecY = vectors(Iy, sY);
    // Y's stride-one index among its free ones, behind C's: gathered in
    // strided vectors where the column split below applies.
    const int yUnit = unit_in(Iy, sY);
    // Column split for tiles of nt columns: the block length f of C's stride-one
    // index placed in front of Y's (0: the whole-index order), and the y set so
    // split in `trial`.
    auto column_block = [&](int nt, std::vector<Index> &trial) -> int64_t {
        if (!maySplit || yUnit <= 0 || Iy[0].strC != 1 || Iy[yUnit].extent % VW ||
            (int)Iy.size() >= kMaxDims)
            return 0;
        // Columns.  A tile then writes C in runs of f elements and reads Y
        // in runs of NT/f elements along v; in the whole-index order it
        // writes runs of up to NT along u and reads Y in runs of NT over
        // the extents before v.  Runs are priced per byte: a read run of
        // L bytes at max(1, 64 / L), a write run at max(1, 128 / L)^2
        // (partial lines are far costlier to write than to read: on
        // MI355X, C runs under 64 bytes slowed the column-split
        // contractions of Appendix A 1.4-3.5x, 32-byte read runs did not).
        // f minimises Y's plus C's price; the whole-index order is kept
        // where it is cheaper (a Y that is small next to C).
        const double Ybytes = itemB * (double)sizeY * (double)an.sizeK;
        const double Cbytes = itemB * (double)sizeX * (double)sizeY;
        auto readPrice = [](double L) { return std::max(1.0, 64.0 / L); };
        auto writePrice = [](double L) {
            const double r = std::max(1.0, 128.0 / L);
            return r * r;
        };
        auto runs = [&](double elems, double cap) { return std::max(1.0, std::min(elems, cap)); };
        double before = 1;
        for (int i = 0; i < yUnit; ++i) before *= (double)Iy[i].extent;
        const double vExt = (double)Iy[yUnit].extent, uExt = (double)Iy[0].extent;
        double best = Ybytes * readPrice(itemB * runs(nt / before, vExt)) +
                      Cbytes * writePrice(itemB * runs(std::min<double>(nt, uExt), uExt));
        int64_t f = 0;
        for (int64_t t = VW; t <= pow2_part(Iy[0].extent) && t * itemB <= 128; t *= 2) {
            if (nt % (t * VW)) continue;
            const double c = Ybytes * readPrice(itemB * runs((double)nt / t, vExt)) +
                             Cbytes * writePrice(itemB * t);
            if (c < best) { best = c; f = t; }
        }
        if (const char *fs = hk.splitF) f = atoi(fs);   // tuning hook
        trial = Iy;
        if (f < VW || (f & (f - 1)) || Iy[0].extent % f || nt % (f * VW)) return 0;
        split_front(trial, 0, (size_t)yUnit, f);
        return aligned(trial, sY, 1) && aligned(Ik, sY, -1) ? f : 0;
    };
    const bool vecC = Iy[0].strC == 1 && Iy[0].extent % VW == 0;
    // C stored in its memory order (see the epilogue below): the run of C along
    // y, when it is shorter than a cache line and a row index continues it in
    // memory; the x index that does.
    const int64_t shortRun =
        Iy[0].strC == 1 && Iy[0].extent * (int64_t)itemB < 128 ? Iy[0].extent : 0;
    auto row_next = [&](const std::vector<Index> &X) {
        for (size_t i = 0; i < X.size() && shortRun; ++i)
            if (X[i].strC == shortRun) return (int)i;
        return -1;
    };
    // whether a tile's plan moves that index to the front of the x order, and
    // what the row operand then gathers
    auto rows_move = [&](const TileShape &c) {
        return row_next(Ix) >= 0 && c.corder && bytesX * 8.0 < bytesC &&
               !(flags & GETT_FLAG_SCALAR);
    };
    const bool vecXMoved = row_next(Ix) >= 0 && vecX &&
                           (sX(Ix[row_next(Ix)]) == 1 || (kvec_ok(sX) && aligned(Ix, sX, -1)));
    // whether C may be accessed in 16-byte vectors, and whole runs of it stored
    // in their memory order (the run's length, 0: not) by a tile's macro-kernel
    auto c_vectors = [&](const TileShape &c) {
        if ((flags & GETT_FLAG_SCALAR) || Iy[0].strC != 1 || Iy[0].extent % VW || c.ry != VW)
            return false;
        for (auto &x : Ix) if (x.strC % VW) return false;
        for (size_t i = 1; i < Iy.size(); ++i) if (Iy[i].strC % VW) return false;
        return true;
    };
    auto c_run = [&](const TileShape &c) -> int64_t {
        const int64_t E = Iy[0].extent;
        const int64_t cap = (int64_t)c.nbuf * c.kt * ((c.mt + VW) + (c.nt + VW));
        if (!c.corder || Iy.size() < 2 || !c_vectors(c) || row_next(Ix) < 0 || E % VW ||
            E >= c.nt || (cap / c.mt - VW) / E < 1)
            return 0;
        return E;
    };
    // Partial tiles (K slices, stream-K tail) are summed through the
    // workspace: the stream of partial tiles and one workgroup's reads of a
    // tile's pieces are priced at these rates (MI355X).
    constexpr double kPartialBw = 5.0e12, kSumBw = 1.0e11;
    // C's run along y: the leading y indices that follow one another in C
    int64_t cRunY = 0;
    if (!Iy.empty() && Iy[0].strC == 1) {
        cRunY = Iy[0].extent;
        for (size_t i = 1; i < Iy.size() && Iy[i].strC == cRunY; ++i) cRunY *= Iy[i].extent;
    }
    // The K box (and whether the K split applies) per box depth, and the column
    // block per tile width: found once, priced for many tiles.
    struct Ahead {
        int kt;
        bool split;
        Box box;
    };
    std::vector<Ahead> aheads;
    aheads.reserve(16);
    auto ahead_for = [&](int kt) -> const Ahead & {
        for (const Ahead &a : aheads)
            if (a.kt == kt) return a;
        std::vector<Index> ksplit;
        const bool split = k_split(kt, ksplit) > 0;
        aheads.push_back({kt, split, split ? box_on(ksplit, 1, kt) : box_for(kt)});
        return aheads.back();
    };
    std::vector<std::pair<int, int64_t>> blocks;
    auto block_for = [&](int nt) {
        for (const auto &b : blocks)
            if (b.first == nt) return b.second;
        std::vector<Index> split;
        blocks.push_back({nt, column_block(nt, split)});
        return blocks.back().second;
    };
    // The longest chain a candidate may sum in and still rank ahead (below),
    // and whether its partial tiles have to fit the fixed workspace.
    double maxChain = std::numeric_limits<double>::infinity();
    bool mustFit = false, inPieces = false;
    auto keeps = [&](const Candidate &c) { return c.chain <= maxChain && (c.fits || !mustFit); };
    auto fits = [](double slotBytes, double counters) {
        return slotBytes <= (double)kFixedSlotBytes && counters <= (double)kFixedCounters;
    };
    auto better = [&](const Candidate &a, const Candidate &b) {
        if (b.tile < 0 || keeps(a) != keeps(b)) return b.tile < 0 || keeps(a);
        return a.cost < b.cost;
    };
    // Every (tile, kernel kind) pair is a candidate; the model ranks them,
    // either by what they cost with the gathers the operands allow (`gathers`)
    // or, for the reference below, as if every tile gathered alike.
    auto candidates = [&](bool gathers) {
    std::vector<Candidate> ranked;
    ranked.reserve(64);
    for (int t = 0; t < num_tiles(dtype); ++t) {
        const TileShape &c = tile_shape(dtype, t);
        if (!gathers && c.nt >= 8 * c.mt) continue;   // the tile for few rows: by its gathers only
        const int64_t block = gathers && !vecY && yUnit > 0 ? block_for(c.nt) : 0;
        const bool vecYSplit = block > 0;
        const double tileBytes = (double)c.mt * c.nt * itemB;
        // a one-box tile is ranked only for a contracted set in one box whose
        // operands are both gathered in vectors: it waits for each operand's
        // gathers in turn, which element-wise gathers make long (it still
        // runs any plan it is forced onto)
        if (c.onebox &&
            (box_for(c.kt).nsteps > 1 || slowGather || (gathers && !(vecX && vecY))) &&
            !(ft && atoi(ft) == t) && !(force && force->tile == t))
            continue;
        const Ahead &ahead = ahead_for(c.kt);
        const bool kSplitAhead = ahead.split;
        const Box &b = ahead.box;
        const double tx = (double)((sizeX + c.mt - 1) / c.mt);
        const double ty = (double)((sizeY + c.nt - 1) / c.nt);
        // What the plan does for C's order: whole runs per tile (the last columns
        // idle, 16 of 128 for runs of 28) and X's vectors lost to the x order
        // (28 x 20 x 20 x 24 x 20 x 20 fp32 over 192 / 256: 526 / 676 us on the
        // 112 columns of 128 x 128 x 16 where 439 / 540 were to be had).
        const int64_t run = gathers && !vecYSplit ? c_run(c) : 0;
        const double tyRun =
            run > 0 ? std::ceil((double)sizeY / (double)(c.nt / run * run)) : ty;
        // Stored by the lanes of the MFMA layout, such a C is partial lines all:
        // 430 MB in runs of 112 bytes took 360 us on 256 x 128.
        const double cutC =
            gathers && dtype == GETT_FLOAT32 && shortRun > 0 && row_next(Ix) >= 0 ? 3.6 : 1.0;
        const bool vecXHere = gathers && rows_move(c) && !vecYSplit ? vecXMoved : vecX;
        // Busiest SIMD: a workgroup of four or more wavefronts is spread over
        // the four SIMDs of one CU (ceil(w / 4) on the busiest), so a CU's
        // load is counted in workgroups; smaller workgroups share SIMDs.
        const int wpt = c.wm * c.wn;
        const double waves = tx * ty * wpt;
        // The busiest CU's tiles pass through its resident slots (cu_time):
        // a last round with fewer tiles than slots leaves wavefronts alone.
        auto per_simd = [&](double tiles) {
            return wpt >= 4 ? cu_time((int)tail_occupancy(c, itemB),
                                      (int)std::ceil(tiles / 256.0), 1.0, 0, 0.0) *
                                  std::ceil(wpt / 4.0)
                            : std::ceil(tiles * wpt / 1024.0);
        };
        const double perSimdRun = per_simd(tx * ty);
        const double kpad = (double)std::max<int64_t>(b.nsteps, 1) * c.kt;
        const double oneChain = (double)an.sizeK;
        const double waveFlops = (double)(c.mt / c.wm) * (c.nt / c.wn) * kpad * 2.0;
        // A K split gathers both operands in 16-byte runs whose cache lines
        // return late: a single LDS buffer waits for them (1.4), and so does a
        // tile with one wavefront per SIMD (1.7: on the fp32 4D x 4D
        // contractions 28 and 30 of Appendix A the 128 x 128 x 32 tile took
        // 17.7 ms, the 128 x 256 x 32 tile with two wavefronts per SIMD
        // 10.5 ms), and the more so a box of 16 fp32 positions, 16-byte runs
        // of both operands (the same contractions: over 21 ms on 128 x 128 x 16).
        const double kSplitWait =
            !kSplitAhead || b.nsteps <= 1                      ? 1.0
            : c.nbuf == 1                                      ? 1.4
            : gathers && dtype == GETT_FLOAT32 && c.kt <= 16 ? 2.2
            : c.wpe == 1                                       ? 1.7
                                                               : 1.0;
        // Element-wise gathers cost an fp32 macro-kernel's one or two
        // wavefronts per SIMD this much of their MFMA rate (odd extents
        // against even ones: 4096^3-shaped 1.1-1.25, C of 529 x 3721 over 3721
        // 1.45 on 32 x 64 tiles).
        // (an X of few rows is a small part of every tile's gathers)
        const bool xVec = vecXHere || (sizeX <= 64 && 16.0 * bytesX < bytesY + bytesC);
        const bool elements =   // some operand's
            gathers && (slowGather || !(xVec && (vecY || vecYSplit || kSplitAhead)));
        const bool both = !vecXHere && !vecY && !vecYSplit;   // both operands'
        const double kElementWise = !gathers || dtype != GETT_FLOAT32 ||
                                            (xVec && (vecY || vecYSplit)) || kSplitAhead
                                        ? 1.0
                                    : c.mt * c.nt <= 32 * 64 ? 1.3
                                    : c.wpe == 1             ? 1.2
                                                             : 1.1;
        // Operands stride-one along different contracted indices that refuse
        // the split: one of them takes another cache line per element, the
        // more boxes, the more often (fp32, 53 x 51 x 50 x 49 over 47 x 45:
        // 128 x 128 x 16 tiles 810 us, 256 x 128 x 32 element-wise 554).
        const bool crossed = gathers && !kSplitAhead && splitXK >= 0 && splitYK >= 0 && splitXK != splitYK;
        const double kCrossed = crossed && dtype == GETT_FLOAT32 && c.kt <= 16 ? 2.0 : 1.0;
        const double tMfma =
            perSimdRun * waveFlops / (peakSimd * c.eff) * kSplitWait * kElementWise * kCrossed;
        // A tile's offset tables, first gathers and C stores, per round of
        // workgroups as measured, and what the first round adds to the launch
        // that every candidate has: 2 us more on the larger tiles of four
        // wavefronts than on the small ones; on those of eight (one workgroup
        // per CU) the round's figure holds it and 0.7 us of the launch.  One
        // workgroup per CU stores C element by element at nearly half the rate
        // of two.
        auto set_up = [&](bool pair) {
            if (!gathers || c.setup <= 0.0f) return 0.0;
            const double us = vecC ? c.setup : c.setupE * (pair ? 0.6 : 1.0);
            return (us * std::ceil(tx * ty / (wpt >= 4 ? 256.0 : 1024.0)) +
                    (wpt >= 8 ? -0.7 : c.mt * c.nt > 2048 ? 2.0 : 0.0)) * 1e-6;
        };
        const double rest = gathers && c.rest > 0.0f && !kSplitAhead ? c.rest : 1.0;
        // Y's lanes run along a free index that Y is not stride-one along: every
        // element comes from a cache line of its own, 0.13-0.19e12 of them a
        // second on every tile and kernel that fills the CUs (each row of tiles
        // reads all of Y again; 136 x 197 x 56 fp32 over 176: 54 us on tiles of 32
        // rows, 32 on 64).  Where the lane order groups the columns by a first
        // index shorter than the tile, up to twice as many.  In fp64 only where whole
        // tiles leave CUs idle, the one place where it was measured to decide
        // (120 x 109 x 7 over 128: 22.9 us on 109 tiles of 32 x 64, 13.3 on 218 of
        // 64 x 32).
        const double group = (double)c.nt / (double)std::max<int64_t>(Iy[0].extent, 1);
        const bool grouped = group >= 1.0 && (4.0 * bytesY >= bytesC || yUnit == 1);
        const double apartRate = 1.0e12 * (0.17 + (grouped ? 0.024 * group : 0.0)) *
                                 (c.nt >= 256 ? 0.8 : 1.0);
        auto apart = [&](double wgs) {
            const double share = std::min(1.0, std::max(wgs, 1.0) * wpt / 1024.0);
            if (!gathers || (dtype != GETT_FLOAT32 && share == 1.0) || vecY || vecYSplit ||
                yUnit < 1)
                return 0.0;
            return (double)sizeY * (double)an.sizeK * tx / (apartRate * share);
        };
        const double tApart = apart(tx * ty);
        // The persistent streaming kernel needs the contracted set in one box.
        const bool canStream = c.stream && b.nsteps <= 1;
        // A stream carried by fewer workgroups than CUs gets that share of the
        // bandwidth (each CU's memory pipeline has its own limit).
        const double cuShare = std::min(1.0, std::max(tx * ty, 1.0) / 256.0);
        // Latency chain: a wavefront walks its K boxes one after another and
        // waits about 1.2 us for each box's gathers when nothing else covers
        // them (measured on MI355X with one wavefront per SIMD); the busiest
        // SIMD walks perSimd wavefronts' boxes, up to four of them resident
        // and waiting together.
        auto chain = [&](double wgs, double boxes) {
            const double ps = std::max(1.0, wpt >= 4 ? std::ceil(wgs / 256.0) * std::ceil(wpt / 4.0)
                                                     : std::ceil(wgs * wpt / 1024.0));
            return ps * boxes * 1.2e-6 / std::min(ps, 4.0);
        };
        const double tChain = chain(tx * ty, (double)std::max<int64_t>(b.nsteps, 1));
        // the larger of throughput and latency bound, with near-ties broken
        // by the other (a 4-norm)
        auto bound = [](double tput, double lat) {
            const double a = tput * tput, b = lat * lat;
            return std::sqrt(std::sqrt(a * a + b * b));
        };
        // Bytes of the stream, C's counted `cut` times.  (A candidate's tMem counts
        // them once: whether C's stream bounds it decides the walk below.)
        auto bytes = [&](double cut) {
            return bytesC * cut + bytesX + bytesY +
                   0.05 * (bytesX * (ty - 1) + bytesY * (tx - 1));
        };
        for (int k = 0; k < (canStream ? 2 : 1); ++k) {
            const double bwFrac = (k ? c.sbw : c.bw) * cuShare;
            // compulsory bytes (each operand read once, C written once) plus
            // the operand panels re-read by other tiles, mostly from L2
            // A single LDS buffer does not overlap the boxes of an fp64 stream
            // (C of 24 x 373248 over 72: 82 us on 64 x 128, 60 on 32 x 64).
            const double cut = k == 0 && run > 0 ? 1.0 : cutC;
            const double tMem = bytes(cut) / (8.0e12 * bwFrac) *
                                (!gathers || dtype != GETT_FLOAT64      ? 1.0
                                 : c.nbuf == 1 && b.nsteps > 1          ? 1.4
                                 : elements && c.mt * c.nt <= 32 * 64 ? 1.25
                                                                      : 1.0);
            Candidate cd;
            cd.tile = t;
            cd.kind = k;
            const double idle = run > 0 && k == 0 ? (double)c.nt / (double)(c.nt / run * run) : 1.0;
            cd.tMfma = idle > 1.0 ? tMfma * per_simd(tx * tyRun) / perSimdRun : tMfma;
            cd.tMem = tMem * idle / bytes(cut) * bytes(1.0);
            // element-wise gathers into a single LDS buffer (the streaming
            // kernel too) wait with nothing to overlap them, as in the K split
            // (the fp32 tiles 256 wide carry sixteen such loads per thread and
            // box: 2.2, 1.7 with more workgroups per CU on 32 rows; one
            // wavefront alone on 64 x 64 1.5)
            const double single =
                !gathers ? (slowGather && (c.nbuf == 1 || k == 1) ? 1.4 : 1.0)
                : !elements                                           ? 1.0
                : c.nbuf == 1 || k == 1                               ? 1.4
                // a column split into single vectors writes C in 16-byte runs
                // (268 x 256 x 16 over 280 fp32: 42 us 256 wide, 31 on 32 x 64)
                : slowGather && xVec && vecYSplit
                    ? (c.nt < 256 ? 1.0 : block <= VW ? 1.6 : 1.4)
                : dtype == GETT_FLOAT32 && c.nt == 256 && c.kt == 16 && !(vecY || vecYSplit)
                    ? (c.mt == 32 ? 1.15 : 1.45)
                : dtype == GETT_FLOAT32 && wpt == 1                   ? 1.15
                                                                      : 1.0;
            cd.chain = oneChain;
            // a stream covers three quarters of the set-up of its tiles
            const double setup = set_up(false);
            const double restHere = run > 0 && k == 0 ? std::max(rest, 0.95) : rest;
            cd.cost = bound(std::max({cd.tMfma * single * restHere + setup,
                                      tMem * idle * single + 0.25 * setup, tApart}),
                            tChain);
            ranked.push_back(cd);
        }
        // Direct-load kernel (tiles that carry it): both operands gathered in
        // vectors.  It sustains deff of the MFMA peak where the macro-kernel
        // sustains eff; its memory stream is priced as the macro-kernel's.
        // After a K split X runs along its block and Y's strided vectors
        // along theirs; nothing is staged in registers, so the split's late
        // lines cost no wait beyond the copy's (kSplitWait).
        if (c.deff > 0.0f && !(flags & GETT_FLAG_SCALAR) && b.nsteps >= 1 &&
            (!gathers      ? !slowGather && !kSplitAhead
             : kSplitAhead ? aligned(Ix, sX, -1)
                           : vecXHere && vecY)) {
            const double tMem = bytes(cutC) / (8.0e12 * c.bw * cuShare);
            Candidate cd;
            cd.tile = t;
            cd.kind = 4;
            cd.chain = oneChain;
            cd.tMfma = tMfma / kSplitWait * c.eff / c.deff *
                       (gathers ? (kSplitAhead ? 1.12 : 1.11) : 1.0);
            cd.tMem = tMem / bytes(cutC) * bytes(1.0);
            cd.cost = bound(std::max(cd.tMfma + set_up(wpt < 8), tMem + 0.25 * set_up(wpt < 8)),
                            tChain);
            ranked.push_back(cd);
        }
        // The same kernel with element-wise copies, for operands that do not
        // both gather in vectors (fp32): the boxes run over the linearised
        // contracted set, so only the last one is padded, and offsets within
        // an operand take 32 bits.
        if (gathers && c.deff > 0.0f && dtype == GETT_FLOAT32 && !(vecX && vecY) &&
            !kSplitAhead && !an.emptySum && an.sizeK < INT32_MAX / 2 && an.maxOffA < INT32_MAX &&
            an.maxOffB < INT32_MAX) {
            const double tMem = bytes(cutC) / (8.0e12 * c.bw * cuShare);
            const double boxes = std::ceil((double)an.sizeK / c.kt);
            Candidate cd;
            cd.tile = t;
            cd.kind = 6;
            cd.chain = oneChain;
            cd.tMfma = tMfma * boxes * c.kt / kpad / kElementWise * c.eff /
                       (wpt >= 8 ? 0.80 : 0.75) * (crossed && c.mt < 256 ? 1.4 : 1.0);
            cd.tMem = tMem / bytes(cutC) * bytes(1.0);
            cd.cost = bound(std::max({cd.tMfma + set_up(wpt < 8), tMem + 0.25 * set_up(wpt < 8),
                                      tApart}),
                            chain(tx * ty, boxes));
            ranked.push_back(cd);
        }
        // Persistent direct-load kernel (tiles that carry it): a contracted
        // set in one box, both operands gathered in vectors; its C stream is
        // priced at dsbw of the HBM peak when C's rows along y run at least a
        // tile wide, else as the macro-kernel's (short runs: measured 1-7%
        // slower than the macro-kernel on the fp64 6D contractions of
        // Appendix A whose y set leads with one index of 24, 3-5% faster
        // on those whose y set leads with a merged run of 384).
        if (c.dsbw > 0.0f && (gathers ? vecX && vecY : !slowGather) && !kSplitAhead &&
            b.nsteps == 1) {
            const double dbw = cRunY >= c.nt ? c.dsbw : c.bw;
            const double tMem = (bytesC + bytesX + bytesY +
                                 0.05 * (bytesX * (ty - 1) + bytesY * (tx - 1))) /
                                (8.0e12 * dbw * cuShare);
            Candidate cd;
            cd.tile = t;
            cd.kind = 5;
            cd.chain = oneChain;
            cd.tMfma = tMfma;
            cd.tMem = tMem;
            cd.cost = bound(std::max(tMfma, tMem), tChain);
            ranked.push_back(cd);
        }
        // K slices: when a contracted set of many boxes meets too few tiles to
        // give every SIMD two wavefronts, P workgroups share each tile's
        // boxes.  Their partial tiles go to the workspace and are summed in
        // slice order by the last of a tile's slices to finish (on the
        // direct-load kernel: by a second launch).  Priced
        // like the macro-kernel on tiles * P workgroups with ceil(boxes / P)
        // boxes each plus two boxes' worth of set-up and epilogue per
        // workgroup, plus the partial tiles' traffic, which adds to the time:
        // P tile writes and reads per tile as a stream, and the last slice's
        // P reads of one tile in turn.  Each slice keeps at least eight
        // boxes.
        if (!(flags & GETT_FLAG_WHOLE_TILES) && !an.emptyC && waves < 2048.0 &&
            b.nsteps >= 16) {
            Candidate best;
            best.tile = -1;
            // Tiles that carry the direct-load kernel slice on it (both operands
            // in vectors): its MFMA rate, the slots summed by a second launch
            // (6 us), as many slices as fill the workgroups the CUs hold at
            // once (two of 128 x 128, one of eight wavefronts), or two or three
            // times that many (shorter chains).  A C of 384 x 376 over 144384:
            // 336 us in 56 slices, 9.1e-7 of the result's norm; 342 us in 113,
            // 6.5e-7; 364 us in 226, 4.7e-7 (32 x 64 tiles of the macro-kernel
            // in 64: 431 us, 8.6e-7).
            const bool directSlices =
                gathers && c.deff > 0.0f && vecXHere && vecY && !kSplitAhead;
            int counts[24], ncounts = 0;
            for (int P = 2; P <= 256; P *= 2) {
                counts[ncounts++] = P;
                if (gathers && inPieces && P < 256) counts[ncounts++] = P + P / 2;
            }
            if (directSlices) {
                const double resident = wpt >= 8 ? 256.0 : 512.0;
                if (resident / (tx * ty) >= 2.0)
                    for (int fill = 1; fill <= 3; ++fill)
                        counts[ncounts++] = (int)(fill * resident / (tx * ty));
            }
            for (int i = 0; i < ncounts; ++i) {
                const int P = counts[i];
                if (b.nsteps / P < 8) continue;
                const double wgs = tx * ty * P;
                const double perSimdP = per_simd(wgs);
                const double kpadP = (std::ceil((double)b.nsteps / P) + 2.0) * c.kt;
                const double tM = perSimdP * (double)(c.mt / c.wm) * (c.nt / c.wn) * kpadP * 2.0 /
                                  (peakSimd * (directSlices ? c.deff : c.eff)) *
                                  (kSplitAhead && c.nbuf == 1 ? 1.4 : 1.0);
                const double shareP = std::min(1.0, wgs / 256.0);
                const double tMemP = (bytesC + bytesX + bytesY +
                                      0.05 * (bytesX * (ty - 1) + bytesY * (tx - 1))) /
                                     (8.0e12 * c.bw * shareP);
                const double tPart =
                    tx * ty * tileBytes * 2.0 * P / kPartialBw +
                    (directSlices ? 6.0e-6 : P * tileBytes / kSumBw + 1.0e-6);
                const double tChainP = chain(wgs, std::ceil((double)b.nsteps / P));
                Candidate cd;
                cd.tile = t;
                cd.kind = 2;
                cd.slices = P;
                // (the sum of the direct-load kernel's slots adds up eight at a time)
                cd.chain = oneChain / P + (directSlices ? std::min(P, 8) + P / 8 : P);
                cd.fits = fits(tx * ty * P * tileBytes, tx * ty);
                cd.tMfma = tM;
                cd.tMem = tMemP;
                // (3, 6, .. 192 slices keep a chain or the workspace's limit that
                // powers of two may not; they take longer than priced: 66 x 72 over
                // 5184 fp64 26.9 us in 48, 22.4 in 32)
                cd.cost = (bound(std::max({tM, tMemP, dtype == GETT_FLOAT32 ? apart(wgs) : 0.0}),
                                 tChainP) + tPart) *
                          (!directSlices && (P & (P - 1)) ? 1.25 : 1.0);
                if (better(cd, best)) best = cd;
            }
            // (element-wise gathers wait in turn into one LDS buffer; in fp32
            // measured 1.1-1.2 times the model's time, on 128 x 128 x 32
            // 1.2-1.6)
            if (elements && !kSplitAhead)
                best.cost *= c.nbuf == 1                              ? (both ? 1.5 : 1.15)
                             : dtype != GETT_FLOAT32                  ? 1.0
                             : c.nt == 256 && c.kt == 16 && c.mt < 64 ? 1.25
                             : crossed                                ? 1.0
                             : c.wpe == 1 && c.kt == 32               ? 1.35
                                                                      : 1.15;
            if (best.tile >= 0) ranked.push_back(best);
        }
        // Stream-K tail: when the tiles do not fill the CUs a whole number of
        // times, the CUs that get one tile more set the time, and a wavefront
        // left alone on its SIMD runs slower than two together.  Instead, the
        // tiles of the complete rounds of G = 256 g workgroups run whole and
        // the boxes of the remaining ones are dealt in equal runs to G more
        // workgroups (g = 1 .. the tile's occupancy; the best is kept); the
        // pieces of a tile shared by several of them are summed through the
        // workspace in piece order by the last to finish.  Priced by cu_time
        // for the busiest CU (two boxes of set-up per piece), the partial
        // tiles' traffic (about r + G tile-sized writes and reads, which add
        // about the time of a 6.8 TB/s stream: measured on MI355X, where they
        // overlap the MFMAs of other workgroups) and the last piece's reads of
        // its tile's pieces.
        const double ntile = tx * ty;
        if (c.tail && !(flags & GETT_FLAG_WHOLE_TILES) && !an.emptyC && wpt >= 4 &&
            b.nsteps >= 16 && ntile > 256.0 && std::fmod(ntile, 256.0) > 0.0) {
            const int occ = (int)tail_occupancy(c, itemB);
            const double boxFlops = (double)(c.mt / c.wm) * (c.nt / c.wn) * c.kt * 2.0;
            const double boxTime =
                std::ceil(wpt / 4.0) * boxFlops / (peakSimd * c.eff) *
                (gathers ? kSplitWait : kSplitAhead && c.nbuf == 1 ? 1.4 : 1.0) * kElementWise *
                kCrossed * (elements && c.nbuf == 1 ? (both ? 2.5 : 1.25) : 1.0);   // spills (element-wise gathers in the
                                                         // piece loop: 869 against 339 us on a C
                                                         // of 529 x 3721 over 3721)
            const double tMem = (bytesC + bytesX + bytesY +
                                 0.05 * (bytesX * (ty - 1) + bytesY * (tx - 1))) /
                                (8.0e12 * c.bw);
            Candidate best;
            best.tile = -1;
            for (int g = 1; g <= occ; ++g) {
                const TailShape ts = tail_shape((int64_t)ntile, b.nsteps, 256 * (int64_t)g);
                const double pieces = std::ceil((double)ts.len / b.nsteps) + 1.0;
                const double units = cu_time(occ, (int)std::ceil(ts.full / 256.0), (double)b.nsteps,
                                             (int)std::ceil(ts.wgs / 256.0),
                                             (double)ts.len + 2.0 * pieces);
                const double tM = units * boxTime;
                const double tPart = (double)(ntile - ts.full + ts.wgs) * tileBytes * 2.0 / 6.8e12 +
                                     pieces * tileBytes / kSumBw + 1.0e-6;
                Candidate cd;
                cd.tile = t;
                cd.kind = 3;
                cd.slices = 256 * g;
                cd.chain = (ts.full + (ntile - ts.full) * tail_chain(ts.len, b.nsteps)) / ntile *
                           oneChain;
                cd.fits = fits(((double)ts.wgs + ntile - (double)ts.full - 1.0) * tileBytes,
                               ntile - (double)ts.full);
                cd.tMfma = tM;
                cd.tMem = tMem;
                cd.cost = bound(std::max({tM, tMem, tApart}), tChain) + tPart;
                if (better(cd, best)) best = cd;
            }
            if (best.tile >= 0) ranked.push_back(best);
        }
    }
    return ranked;
    };
    // Ties (the same estimate to 0.01 us: mirror-image tiles on a square
    // problem) between tiles of at least 64 x 64 go to the one wider along y,
    // whose C runs are longer (measured on MI355X: fp64 64 x 128 x 24 against
    // 128 x 64 x 24 on the 4D x 4D contractions of Appendix A, 1-4% faster);
    // small tiles keep the table's order (fp32 64 x 32 was 3-5% faster than
    // 32 x 64 on the latency-bound points of Fig. 11).
    auto wideY = [&](const Candidate &c) {
        const TileShape &t = tile_shape(dtype, c.tile);
        return t.mt >= 64 && t.nt >= 64 ? t.nt : 0;
    };
    auto cheaper = [&](const Candidate &a, const Candidate &b) {
        const long long ka = llround(a.cost * 1e8), kb = llround(b.cost * 1e8);
        if (ka != kb) return ka < kb;
        return wideY(a) > wideY(b);
    };
    // The reference: the cheapest candidate of the model without the cost of
    // gathers.  That cost moves the choice between kernels; it must not move
    // what a caller gets, so a candidate that sums in longer chains than the
    // reference ranks behind the cheapest that does not (the rounding error of
    // a sum grows as the square root of its chain: fp32, measured at contracted
    // sets of 2160 to 144384 in 1 to 256 slices, 1.79e-8 of the result's norm
    // times the square root of the positions per slice plus the slices, within
    // 2%; a tail's 947 against 937), and so does
    // one that gett_contract_noalloc would refuse where it takes the reference.
    // The reference itself is ranked when no other candidate keeps to it.
    const std::vector<Candidate> plain = candidates(false);
    const Candidate ref = *std::min_element(plain.begin(), plain.end(), cheaper);
    maxChain = ref.chain * (1.0 + 1e-9);
    mustFit = ref.fits;
    inPieces = ref.kind == 2 || ref.kind == 3;
    std::vector<Candidate> ranked = candidates(true);
    if (std::none_of(ranked.begin(), ranked.end(), keeps)) ranked.push_back(ref);
    // A twentieth between two prices decides nothing, so the reference's is
    // reduced by that much (a direct-load kernel that its operands refuse runs
    // as its tile's macro-kernel).  Over 931 measured contractions the plans take
    // 0.778 of the time they took without the price of gathers, and 12 of them
    // more than 1.04; without the reduction about 1.6 times as many do.
    auto stays = [&](int kind) {
        for (Candidate &c : ranked)
            if (c.tile == ref.tile && c.kind == kind) {
                c.cost *= 0.95;
                return true;
            }
        return false;
    };
    if (!stays(ref.kind) && ref.kind >= 4) stays(0);
    double first = std::numeric_limits<double>::infinity();
    for (const Candidate &c : ranked)
        if (keeps(c)) first = std::min(first, c.cost);
    for (Candidate &c : ranked)
        if (!keeps(c)) c.cost = std::max(c.cost, 1.01 * first);
    std::stable_sort(ranked.begin(), ranked.end(), cheaper);
    Candidate pick = ranked[0];
    const char *how = "model";
    auto find = [&](int t, int k) -> const Candidate * {
        for (auto &c : ranked)
            if (c.tile == t && c.kind == k) return &c;
        return nullptr;
    };
    // tuning and test hooks; a choice being timed by gett_plan_tune overrides
    // them, a remembered one does not
    if (force && (force->timing || !(ft || fk))) {
        if (const Candidate *c = find(force->tile, force->kind)) {
            pick = *c;
            how = force->source;
        }
    } else if (ft || fk) {
        const int t = ft ? atoi(ft) : pick.tile;
        const int k = fk ? atoi(fk) : 0;
        const Candidate *c = find(t, k);
        if (!c) c = find(t, 0);
        if (c) {
            pick = *c;
            how = "forced";
            // the stream-K tail on any plan of a tile that carries it (the
            // model ranks it only where it may pay)
            if (k == 3 && c->kind == 0 && tile_shape(dtype, t).tail && !an.emptyC &&
                !(flags & GETT_FLAG_WHOLE_TILES))
                pick.kind = 3;
        }
    }
    // tuning hook: this many K slices on the chosen tile
    // (1: none), unless the plan must be deterministic
    if (const char *fs = hk.forceKslices) {
        const int P = atoi(fs);
        if (P == 1 && pick.kind == 2) {
            if (const Candidate *c = find(pick.tile, 0)) pick = *c;
        } else if (P > 1 && pick.kind != 1 && !an.emptyC && !(flags & GETT_FLAG_WHOLE_TILES)) {
            pick.kind = 2;
            pick.slices = P;
        }
    }
    const int tile = pick.tile;
    int kind = pick.kind;
    const int kslices = kind == 2 ? pick.slices : 1;
    const double bestMfma = pick.tMfma, bestMem = pick.tMem;
    const TileShape &ts = tile_shape(dtype, tile);

    // ---- index splitting (Sec. 3.2.1, Fig. 5: the sub-tensors keep the
    //      stride-one index of every tensor; Examples 1-2: one index read as
    //      two).  The tiles are linear ranges of each set in its order, so a
    //      set whose first index is one tensor's stride-one index and whose
    //      second is another's holds both runs only when the first is
    //      blocked: (u, v, ...) becomes (u_in, v, u_out, ...) with u_in of
    //      extent f.  Two cases:
    //        columns -- C's stride-one index u and the column operand's
    //                   stride-one index v are different free indices of
    //                   the column set: C is written in runs of f elements,
    //                   Y is read in 16-byte vectors along v;
    //        K box   -- the row operand's stride-one index u and the column
    //                   operand's v are different contracted indices: X is
    //                   read in vectors along u_in, Y along v.
    //      f is a power of two dividing S_u; the vectors of Y then gather
    //      elements f rows (K positions) apart. ----
    int ysplit = 0;   // 0, kGatherRowVecStrided or kGatherKVecStrided
    int yes = 1;
    if (maySplit) {
        // which set holds each operand's stride-one index
        const int yRow = unit_in(Iy, sY);
        std::vector<Index> trial;
        if (yRow > 0 && Iy[0].strC == 1 && Iy[yRow].extent % VW == 0 &&
            (int)Iy.size() < kMaxDims) {
            const int64_t f = column_block(ts.nt, trial);
            if (f > 0) {
                Iy.swap(trial);
                ysplit = kGatherRowVecStrided;
                yes = (int)f;
            }
        } else {
            const int64_t f = k_split(ts.kt, trial);
            if (f > 0) {
                Ik.swap(trial);
                nk = (int)Ik.size();
                kvecIdx = 1;
                // the streaming kernel takes the contracted set in one box
                if (kind == 1 && box_for(ts.kt).nsteps > 1) {
                    Ik.swap(trial);
                    nk = (int)Ik.size();
                    kvecIdx = 0;
                } else {
                    ysplit = kGatherKVecStrided;
                    yes = (int)f;
                    if (kind == 4) walk_lines(ts.kt);
                }
            }
        }
    }
    // Y is stride-one along a free index behind C's, but extents or strides
    // refuse the split: taken element by element in C's order, every lane
    // reads another cache line and the rest of it is gone before the tile
    // that needs it.  The index moves up behind C's, where the lanes can walk
    // it (the lane order below) and neighbouring tiles find the lines in L2
    // -- unless Y is so small beside C that it stays there anyway.
    // (47 x 35 x 23 x 33 x 45 fp32 over 34: 1499 us, then 261 to 474 by tile.)
    if (maySplit && !ysplit && !vecY && yUnit > 1 && Iy[0].strC == 1 && 4.0 * bytesY >= bytesC)
        std::rotate(Iy.begin() + 1, Iy.begin() + yUnit, Iy.begin() + yUnit + 1);
    const Box box = box_for(ts.kt);
    // A contraction bound by the C stream walks C in memory order: x indices
    // by C stride (the row operand's stride-one index stays first when it is
    // a free index, for its vector gathers) and tiles y-fastest.
    const bool streaming = bestMem > bestMfma;
    // Where C is stored in its memory order (below), consecutive tile rows have
    // to be consecutive in C: that row index leads the x order -- taken when the
    // row operand is small next to C (its gathers may lose their vectors).
    const int rowNext = row_next(Ix);
    const bool corderRows = ysplit != kGatherRowVecStrided && rows_move(ts);
    if (streaming) {
        std::stable_sort(Ix.begin(), Ix.end(), [](const Index &a, const Index &b) {
            return a.strC < b.strC;
        });
        for (size_t i = 0; i < Ix.size() && !corderRows; ++i)
            if (sX(Ix[i]) == 1) {
                std::rotate(Ix.begin(), Ix.begin() + i, Ix.begin() + i + 1);
                break;
            }
    } else if (corderRows) {
        std::rotate(Ix.begin(), Ix.begin() + rowNext, Ix.begin() + rowNext + 1);
    }
    const int kj = box.kj;
    const int64_t tj = box.tj, kbox = box.kbox, nblk = box.nblk, nsteps = box.nsteps;

    // ---- gather modes ----
    auto row_vec_ok = [&](const std::vector<Index> &I, auto strOf) {
        if (strOf(I[0]) != 1 || I[0].extent % VW) return false;
        for (size_t i = 1; i < I.size(); ++i)
            if (strOf(I[i]) % VW) return false;
        for (auto &k : Ik)
            if (strOf(k) % VW) return false;
        return true;
    };
    auto k_vec_ok = [&](const std::vector<Index> &I, auto strOf) {
        if (!kvec_ok(strOf)) return false;
        if (kj == 0 && (tj % VW)) return false;
        for (auto &x : I)
            if (strOf(x) % VW) return false;
        return true;
    };
    int xmode = kGatherScalar, ymode = kGatherScalar;
    if (!(flags & GETT_FLAG_SCALAR)) {
        if (row_vec_ok(Ix, sX)) xmode = kGatherRowVec;
        else if (k_vec_ok(Ix, sX)) xmode = kGatherKVec;
        if (ysplit) ymode = ysplit;
        else if (row_vec_ok(Iy, sY)) ymode = kGatherRowVec;
        else if (k_vec_ok(Iy, sY)) ymode = kGatherKVec;
    }
    // The direct-load kernel takes vector gathers of both operands; a plan
    // that ends up otherwise runs its tile's macro-kernel.
    if (kind == 4 && !(direct_modes(xmode, ymode) && nsteps >= 1)) kind = 0;
    if (kind == 5 && !(xmode <= kGatherKVec && ymode <= kGatherKVec && nsteps == 1)) kind = 0;
    const bool cvec = c_vectors(ts);
    // C stored in its memory order through LDS (unpack_c_order): when C's
    // stride-one run along y is shorter than a cache line and C continues in
    // memory along a row index, the per-lane stores would cut every line.
    // At least one run must fit a staging pass of the packing buffers.
    int crun = kind == 0 && kslices == 1 && ysplit != kGatherRowVecStrided ? (int)c_run(ts) : 0;
    if (const char *co = hk.cOrder) {   // tuning hook: 0 turns it off
        if (atoi(co) == 0) crun = 0;
    }

    // ---- addressing: the kernels reach each tile through 64-bit base
    //      offsets and address inside it with 32-bit offsets (rows and
    //      columns relative to the tile's base, K-box positions relative to
    //      the box origin), so tensors may hold 2^31 elements or more as long
    //      as one tile's rows plus one box span less than 2^31 - 1 elements.
    //      Over R consecutive positions of a set, digit i moves at most
    //      min(e_i - 1, floor((R - 1) / P_i) + 1) above its lowest value
    //      (P_i: product of the earlier extents). ----
    {
        constexpr int64_t cap = (int64_t)1 << 62;
        auto sat = [](int64_t a, int64_t b) {   // a * b, saturating at cap
            return (a != 0 && b > cap / a) ? cap : a * b;
        };
        auto span = [&](const std::vector<Index> &I, auto strOf, int64_t R) {
            int64_t tot = 0, P = 1;
            for (const Index &x : I) {
                const int64_t moves = std::min<int64_t>(x.extent - 1, (R - 1) / P + 1);
                tot = std::min(cap, tot + sat(std::max<int64_t>(moves, 0), strOf(x)));
                P = sat(P, std::max<int64_t>(x.extent, 1));
            }
            return tot;
        };
        auto kspan = [&](auto strOf) {
            int64_t tot = sat(box.tj - 1, strOf(Ik[box.kj]));
            for (int i = 0; i < box.kj; ++i)
                tot = std::min(cap, tot + sat(Ik[i].extent - 1, strOf(Ik[i])));
            return tot;
        };
        auto sC = [](const Index &x) { return x.strC; };
        const int64_t lim = INT32_MAX;
        if (!an.emptyC && (span(Ix, sX, ts.mt) + kspan(sX) >= lim ||
                           span(Iy, sY, ts.nt) + kspan(sY) >= lim ||
                           span(Ix, sC, ts.mt) + span(Iy, sC, ts.nt) >= lim))
            return GETT_ERROR_NOT_SUPPORTED;
    }

    // ---- descriptor ----
    KDesc d = {};
    auto dim = [](int64_t e, int64_t s0, int64_t s1) {
        return KDim{(int32_t)e, recip(e), 0, s0, s1};
    };
    d.sizeX = sizeX;
    d.sizeY = sizeY;
    d.nx = (int)Ix.size();
    d.ny = (int)Iy.size();
    d.nk = nk;
    if (d.nx + d.ny + d.nk > kMaxIndices) return GETT_ERROR_NOT_SUPPORTED;   // cannot happen
    KDim *at = d.dim;
    for (const Index &i : Ix) *at++ = dim(i.extent, sX(i), i.strC);
    for (const Index &i : Iy) *at++ = dim(i.extent, sY(i), i.strC);
    for (const Index &i : Ik) *at++ = dim(i.extent, sX(i), sY(i));
    d.kj = kj;
    d.tj = (int32_t)tj;
    d.kbox = (int32_t)kbox;
    d.nblk = (int32_t)std::max<int64_t>(nblk, 1);
    d.nblkInv = recip(d.nblk);
    d.linK = kind == 6 ? (int32_t)an.sizeK : 0;
    d.nsteps = nsteps;
    // With C stored in its memory order a tile takes whole runs of C only (240
    // of 256 columns for runs of 24): a run cut by a tile's edge is written in
    // two partial pieces by two workgroups, and a bare stream of stores over
    // such a C (369 MB, runs of 24) takes 97-100 us with cut runs against
    // 74-76 us with whole ones.
    d.stepY = crun > 0 ? ts.nt / crun * crun : ts.nt;
    const int64_t tilesX = (sizeX + ts.mt - 1) / ts.mt;
    const int64_t tilesY = (sizeY + d.stepY - 1) / d.stepY;
    if (!an.emptyC && (tilesX * tilesY * ts.wm * ts.wn * 64 >= (int64_t)UINT32_MAX || sizeX >= INT32_MAX ||
                       sizeY >= INT32_MAX || nsteps >= INT32_MAX))
        return GETT_ERROR_NOT_SUPPORTED;
    d.tilesX = (int32_t)tilesX;
    d.tilesY = (int32_t)tilesY;
    d.group = (int32_t)std::max<int64_t>(1, std::min<int64_t>(8, tilesX));
    d.tilesYInv = recip(tilesY);
    d.bandInv = recip((int64_t)d.group * tilesY);
    d.groupInv = recip(d.group);
    d.order = streaming ? 1 : 0;
    d.xcdremap = -1;   // decided per call (see gett_contract)
    if (const char *xr = hk.xcdRemap) d.xcdremap = atoi(xr) != 0;   // tuning hook
    // element-wise where the caller asks for it; a tile whose lanes do not own
    // VW consecutive columns has no other access
    d.cvec = cvec ? 1 : (flags & GETT_FLAG_SCALAR) || ts.ry != VW ? -1 : 0;
    d.xscalar_kfast = sX(Ik[0]) < sX(Ix[0]) ? 1 : 0;
    d.yscalar_kfast = sY(Ik[0]) < sY(Iy[0]) ? 1 : 0;
    // Element-wise gathers of an operand that is stride-one along the second
    // index of its free set: the lanes walk that index (rows grouped by the
    // first index's value) -- their loads then touch few cache lines.
    auto lane_perm = [&](const std::vector<Index> &I, auto strOf, int mode, int rows,
                         int32_t &kfast) -> int32_t {
        if (mode != kGatherScalar || I.size() < 2 || strOf(I[1]) != 1 || I[0].extent >= rows ||
            I[0].extent < 2)
            return 0;
        kfast = 0;
        return (int32_t)I[0].extent;
    };
    d.xperm = lane_perm(Ix, sX, xmode, ts.mt, d.xscalar_kfast);
    d.yperm = lane_perm(Iy, sY, ymode, ts.nt, d.yscalar_kfast);
    if (const char *lp = hk.lanePerm) {   // tuning hook: 0 turns it off
        if (atoi(lp) == 0) d.xperm = d.yperm = 0;
    }
    d.yes = yes;
    d.kslices = kslices;
    d.crun = crun;
    d.piecesInv = recip(crun / VW);
    d.tile0 = 0;
    d.tailFull = d.tailWgs = d.tailLen = 0;
    if (kind == 3 && !an.emptyC) {
        // the model's number of tail workgroups (256 when the tail was forced
        // on a plan the model did not rank it for; tuning hook: GETT_TAIL_WGS)
        int64_t wgs = pick.kind == 3 && pick.slices > 1 ? pick.slices : 256;
        if (const char *tw = hk.tailWgs) wgs = std::max<int64_t>(1, atoll(tw));
        const TailShape tsh = tail_shape((int64_t)tilesX * tilesY, std::max<int64_t>(nsteps, 1), wgs);
        d.tailFull = (int32_t)tsh.full;
        d.tailWgs = (int32_t)tsh.wgs;
        d.tailLen = (int32_t)tsh.len;
    }
    if (!an.emptyC && tilesX * tilesY * kslices * ts.wm * ts.wn * 64 >= (int64_t)UINT32_MAX)
        return GETT_ERROR_NOT_SUPPORTED;
    // Workspace of the partial tiles: a counter per tile that has pieces and
    // a slot per piece (K slices: every slice of every tile; stream-K tail:
    // slots up to (tail workgroups - 1) + (tail tiles - 1), see the kernel).
    int64_t wsSlots = 0, wsCounters = 0;
    if (!an.emptyC) {
        const int64_t tiles = tilesX * tilesY;
        if (kslices > 1) {
            wsSlots = tiles * kslices;
            wsCounters = tiles;
        } else if (kind == 3) {
            wsCounters = tiles - d.tailFull;
            wsSlots = d.tailWgs + wsCounters - 1;
        }
    }
    plan.wsCounters = (uint64_t)wsCounters;
    plan.wsTileBytes = (uint64_t)wsSlots * ts.mt * ts.nt * (dtype == GETT_FLOAT32 ? 4 : 8);

    plan.dtype = dtype;
    plan.flags = flags;
    plan.hooks = hk.text;
    plan.rank[0] = rank[0];
    plan.rank[1] = rank[1];
    plan.rank[2] = rank[2];
    plan.an = an;
    plan.desc = d;
    plan.descScalar = d;
    plan.descScalar.cvec = 0;
    plan.tile = tile;
    plan.xmode = xmode;
    plan.kind = kind;
    plan.ranked = ranked;
    plan.ymode = ymode;
    const double item = dtype == GETT_FLOAT32 ? 4.0 : 8.0;
    plan.flops = 2.0 * (double)an.sizeM * (double)an.sizeN * (double)an.sizeK;
    const double nA = (double)an.sizeM * an.sizeK, nB = (double)an.sizeN * an.sizeK,
                 nC = (double)an.sizeM * an.sizeN;
    plan.bytesAlgo = item * (nA + nB + nC);

    // ---- description ----
    std::ostringstream o;
    o << "{\"dtype\":\"" << (dtype == GETT_FLOAT32 ? "f32" : "f64") << "\",";
    json_set(o, "I_m", an.Im, true, false, true);
    o << ",";
    json_set(o, "I_n", an.In, false, true, true);
    o << ",";
    json_set(o, "I_k", an.Ik, true, true, false);
    o << ",\"merges\":[";
    for (size_t i = 0; i < an.merges.size(); ++i) o << (i ? "," : "") << "\"" << an.merges[i] << "\"";
    o << "],\"swapped\":" << (swap ? "true" : "false");
    o << ",\"row_operand\":\"" << (swap ? "B" : "A") << "\",\"col_operand\":\"" << (swap ? "A" : "B")
      << "\"";
    auto names = [&](const char *key, const std::vector<Index> &s) {
        o << ",\"" << key << "\":[";
        for (size_t i = 0; i < s.size(); ++i) o << (i ? "," : "") << "\"" << s[i].name << "\"";
        o << "]";
    };
    names("x_order", Ix);
    names("y_order", Iy);
    names("k_order", Ik);
    o << ",\"size_x\":" << sizeX << ",\"size_y\":" << sizeY << ",\"size_k\":" << an.sizeK;
    o << ",\"tile\":{\"id\":" << tile << ",\"mt\":" << ts.mt << ",\"nt\":" << ts.nt << ",\"kt\":" << ts.kt
      << ",\"waves\":[" << ts.wm << "," << ts.wn << "],\"reads\":[" << ts.rx << "," << ts.ry
      << "],\"waves_per_simd\":" << ts.wpe << ",\"prefetch\":" << ts.pf
      << ",\"lds_buffers\":" << ts.nbuf << ",\"one_box\":" << (ts.onebox ? "true" : "false")
      << ",\"c_order_epilogue\":" << (ts.corder ? "true" : "false")
      << ",\"chosen_by\":\"" << how << "\",\"model_us\":" << pick.cost * 1e6 << "}";
    o << ",\"hooks\":\"" << hk.text << "\"";
    auto candidate = [&](const Candidate &c) {
        o << "{\"tile\":" << c.tile << ",\"kind\":\"" << kind_name(c.kind) << "\"";
        if (c.kind == 2) o << ",\"kslices\":" << c.slices;
        if (c.kind == 3) o << ",\"tail_workgroups\":" << c.slices;
        o << ",\"model_us\":" << c.cost * 1e6 << "}";
    };
    o << ",\"candidates\":[";
    for (size_t i = 0; i < ranked.size(); ++i) {
        if (i) o << ",";
        candidate(ranked[i]);
    }
    o << "],\"reference\":";
    candidate(ref);
    o << ",\"chain\":" << pick.chain << ",\"reference_chain\":" << ref.chain
      << ",\"reference_fits\":" << (ref.fits ? "true" : "false");
    o << ",\"streaming\":" << (streaming ? "true" : "false");
    const bool onDirect = kind == 2 && direct_slices(ts.deff > 0.0f, xmode, ymode);
    o << ",\"kernel\":\"" << (onDirect ? "direct" : kind == 2 ? "macro" : kind_name(kind))
      << "\",\"kslices\":" << kslices;
    o << ",\"tail\":{\"full_tiles\":" << d.tailFull << ",\"workgroups\":" << d.tailWgs
      << ",\"boxes\":" << d.tailLen << "}";
    o << ",\"partials\":\"" << (kslices > 1 || kind == 3 ? "workspace" : "none")
      << "\",\"workspace_bytes\":" << plan.wsTileBytes
      << ",\"workspace_counters\":" << plan.wsCounters;
    o << ",\"kbox\":{\"kj\":" << kj << ",\"tj\":" << tj << ",\"elements\":" << kbox << ",\"blocks\":" << nblk
      << ",\"steps\":" << nsteps << "}";
    o << ",\"gather_x\":\"" << mode_name(xmode) << "\",\"gather_y\":\"" << mode_name(ymode)
      << "\",\"c_vector\":" << (cvec ? "true" : "false") << ",\"c_access\":\""
      << (onDirect || d.cvec < 0 ? "element" : d.cvec > 0 ? "vector" : "run") << "\"" << ",\"y_vector_stride\":" << yes
      << ",\"c_order_run\":" << crun << ",\"lane_perm\":[" << d.xperm << "," << d.yperm << "]";
    o << ",\"grid\":{\"tiles_x\":" << tilesX << ",\"tiles_y\":" << tilesY << ",\"workgroups\":"
      << tilesX * tilesY << ",\"threads\":" << ts.wm * ts.wn * 64 << "}";
    o << ",\"empty_c\":" << (an.emptyC ? "true" : "false") << ",\"empty_sum\":"
      << (an.emptySum ? "true" : "false");
    char buf[64];
    snprintf(buf, sizeof buf, "%.17g", plan.flops);
    o << ",\"flops\":" << buf;
    snprintf(buf, sizeof buf, "%.17g", plan.bytesAlgo);
    o << ",\"bytes_min\":" << buf << "}";
    plan.text = o.str();
    return GETT_SUCCESS;
}

}  // namespace gett
