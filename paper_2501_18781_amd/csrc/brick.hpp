// brick.hpp -- the cell-brick work unit shared by the operator kernels.
//
// A 64-thread workgroup (one wavefront) owns a brick of 4x4x4 cells, one
// thread per cell; the brick's 9x9x9 Q2 nodes are staged in LDS.  The heat
// applies use the same cells and node sums in slabs (Slab, below).
//
// Staging of a brick is per node (the lanes stage its 9-node rows; FP64) or, in
// the FP32 diagonal, per cell (each thread reads the 27 nodes of its cell and
// writes them to LDS; nodes shared by cells of the brick are written with
// the same value by each).  Finishing is by ownership: a cell owns its
// local nodes (a, b, c) with a, b, c in {0, 1}, and the last valid cell of
// the brick in a direction also owns the local nodes with index 2 in that
// direction, so every brick node is finished by exactly one thread, with
// fully unrolled code and no index division.  A node's sum runs over the
// cells of the brick that contain it (at most 8) in a fixed order.
//
// A node on a face that a neighbouring brick also touches ("shared") is not
// written to the output: its partial sum goes to the brick's slot in a face
// buffer (one slot per brick node), and a second kernel adds
// the partials of the (2, 4 or 8) bricks that share it, in a fixed order.
// Every output entry is therefore written exactly once, without atomics and
// without clearing the output first, and the result is bitwise reproducible.
//
// Bricks are numbered so that each XCD receives a contiguous range of them
// (workgroups are dispatched to the 8 XCDs round robin), which keeps the
// neighbours that share faces, and their halo loads, in one L2.
#pragma once

#include <type_traits>

#include "kernels.hpp"

namespace mf {

constexpr int BB = 4;               // cells per brick edge
constexpr int BNT = BB * BB * BB;   // threads (cells) per brick
constexpr int BP = 2 * BB + 1;      // nodes per brick edge
constexpr int NXCD = 8;

// LDS layout of a staged brick field: node (lx, ly, lz) at lx + R ly + R BP lz.
// For 8-byte entries the rows are padded to R = 10: a wavefront's gather of
// node (2tx + a, 2ty + b, 2tz + c) then spreads its stride-2 accesses over
// more LDS banks than with R = 9 (FP64 apply kernel 30.0 -> 27.7 us at 64^3,
// Oseen 72.6 -> 68.4 us at 48^3); 4-byte entries keep R = 9 (padding
// measured no faster there).
template <typename T> __host__ __device__ constexpr int lds_row() { return sizeof(T) == 8 ? BP + 1 : BP; }
template <typename T> __host__ __device__ constexpr int lds_plane() { return lds_row<T>() * BP; }
// LDS entries of one staged field
template <typename T> __host__ __device__ constexpr int lds_field() { return lds_plane<T>() * BP; }

constexpr int BNB = BP * BP * BP;            // nodes per brick
constexpr int BFACE = BNB + 2 * BP * BP;     // its face-buffer slots, see face_slot

__host__ __device__ inline int64_t n_bricks(const KMesh &m)
{
    return (int64_t)((m.nx + BB - 1) / BB) * ((m.ny + BB - 1) / BB) * ((m.nz + BB - 1) / BB);
}

// Face-buffer slot of a brick node (only the slots of shared surface nodes
// are ever written or read).  Nodes on the brick's two x faces get a region
// of their own, (side, ly, lz) with ly fastest, so that the combine pass
// reads them in runs along y; every other node keeps its lexicographic brick
// index, so that runs along x stay contiguous.
__host__ __device__ __forceinline__ constexpr int face_slot(int lx, int ly, int lz)
{
    return (lx == 0 || lx == 2 * BB) ? BNB + (lx ? BP * BP : 0) + ly + BP * lz
                                     : lx + BP * (ly + BP * lz);
}

struct Brick {
    static constexpr int NT = BNT, PZ = BP, NNODES = BNB, NFACE = BFACE;
    static constexpr int W = 1, CX = BB; // wavefronts; cells along x
    template <typename T> static __host__ __device__ constexpr int field() { return lds_field<T>(); }
    static __device__ __forceinline__ constexpr int face_slot_of(int lx, int ly, int lz) { return face_slot(lx, ly, lz); }

    int brick;         // natural brick index (x fastest)
    int bx, by, bz;    // brick coordinates
    int c0x, c0y, c0z; // first cell of the brick
    int ncx, ncy, ncz; // valid cells per direction (clipped at the mesh end)
    int t;             // this thread's cell slot within the brick (0..63)
    int tx, ty, tz;    // this thread's cell within the brick
    bool valid;
    bool lastx, lasty, lastz;

    __device__ __forceinline__ Brick(const KMesh &m, int slot) : Brick(m, slot, xcd_index()) {}

    // XCD-contiguous numbering: workgroup b runs on XCD b % 8; XCD k gets
    // the workgroup indices [start_k, start_k + count_k).
    static __device__ __forceinline__ int xcd_index()
    {
        const int G = gridDim.x, q = G / NXCD, r = G % NXCD;
        const int k = blockIdx.x % NXCD, j = blockIdx.x / NXCD;
        return k * q + min(k, r) + j;
    }

    // The brick of natural index b.
    __device__ __forceinline__ Brick(const KMesh &m, int slot, int b) : t(slot)
    {
        brick = b;
        const int nbx = (int)((unsigned)(m.nx + BB - 1) / BB), nby = (int)((unsigned)(m.ny + BB - 1) / BB);
        const int q = (int)udiv((unsigned)brick, (unsigned)nbx, m.rbx);
        bx = brick - q * nbx;
        bz = (int)udiv((unsigned)q, (unsigned)nby, m.rby);
        by = q - bz * nby;
        c0x = bx * BB;
        c0y = by * BB;
        c0z = bz * BB;
        ncx = min(BB, m.nx - c0x);
        ncy = min(BB, m.ny - c0y);
        ncz = min(BB, m.nz - c0z);
        tx = t & (BB - 1);
        ty = (t / BB) & (BB - 1);
        tz = t / (BB * BB);
        valid = tx < ncx && ty < ncy && tz < ncz;
        lastx = valid && tx == ncx - 1;
        lasty = valid && ty == ncy - 1;
        lastz = valid && tz == ncz - 1;
    }

    template <typename T> static __device__ __forceinline__ constexpr int lds_index(int lx, int ly, int lz)
    {
        return lx + lds_row<T>() * ly + lds_plane<T>() * lz;
    }

    // face_slot of this thread's cell node (a, b, c).
    __device__ __forceinline__ int fslot(int a, int b, int c) const
    {
        const int lex = (2 * tx + a) + BP * ((2 * ty + b) + BP * (2 * tz + c));
        if (a == 1) return lex;
        const bool xface = a == 0 ? tx == 0 : tx == BB - 1;
        return xface ? NNODES + (a ? BP * PZ : 0) + (2 * ty + b) + BP * (2 * tz + c) : lex;
    }

    __device__ __forceinline__ int64_t cell_index(const KMesh &m) const
    {
        return (int64_t)(c0x + tx) + (int64_t)m.nx * ((c0y + ty) + (int64_t)m.ny * (c0z + tz));
    }

    // Whether the brick has a node on a Dirichlet face (uniform over the brick).
    __device__ __forceinline__ bool touches_dirichlet(const KMesh &m) const
    {
        const unsigned f = m.dirichlet;
        return ((f & 1u) && c0x == 0) || ((f & 2u) && c0x + ncx == m.nx) || ((f & 4u) && c0y == 0) ||
               ((f & 8u) && c0y + ncy == m.ny) || ((f & 16u) && c0z == 0) || ((f & 32u) && c0z + ncz == m.nz);
    }

    // Neighbours on all six sides (and so no Dirichlet face).
    __device__ __forceinline__ bool inner(const KMesh &m) const
    {
        return bx > 0 && by > 0 && bz > 0 && c0x + BB < m.nx && c0y + BB < m.ny && c0z + BB < m.nz;
    }

    // Visit the nodes this thread owns: f(a, b, c, lds_index, global_index,
    // constrained, shared), with a, b, c compile-time constants and
    // lds_index in the layout of a staged field of T.  `shared` is
    // an int: bit 0 set if a neighbouring brick also touches the node, bit 1
    // if that happens through one of this brick's high faces (the node is
    // then finished by another brick's combine pass).  The eight
    // low nodes of every valid cell come first; the high faces, owned by the
    // last cells, follow in seven groups that each test one uniform flag.
    template <typename T = double, typename F> __device__ __forceinline__ void for_owned_nodes(const KMesh &m, F f) const
    {
        constexpr int R = lds_row<T>(), P = lds_plane<T>();
        if (!valid) return;
        const int gx0 = 2 * (c0x + tx), gy0 = 2 * (c0y + ty), gz0 = 2 * (c0z + tz);
        const int64_t g0 = node_index(m, gx0, gy0, gz0);
        const int64_t sy = m.NX, sz = (int64_t)m.NX * m.NY;
        const int l0 = lds_index<T>(2 * tx, 2 * ty, 2 * tz);
        // Per direction, for local index 0 and 2 (index 1 is never on a
        // boundary or a brick face): Dirichlet flag and shared-face flag.
        const unsigned f6 = m.dirichlet;
        const bool dx0 = (f6 & 1u) && gx0 == 0, dx2 = (f6 & 2u) && gx0 + 2 == m.NX - 1;
        const bool dy0 = (f6 & 4u) && gy0 == 0, dy2 = (f6 & 8u) && gy0 + 2 == m.NY - 1;
        const bool dz0 = (f6 & 16u) && gz0 == 0, dz2 = (f6 & 32u) && gz0 + 2 == m.NZ - 1;
        const bool sx0 = tx == 0 && gx0 > 0, sx2 = gx0 + 2 < m.NX - 1;
        const bool sy0 = ty == 0 && gy0 > 0, sy2 = gy0 + 2 < m.NY - 1;
        const bool sz0 = tz == 0 && gz0 > 0, sz2 = gz0 + 2 < m.NZ - 1;
        auto node = [&](auto A, auto B, auto C) {
            constexpr int a = decltype(A)::value, b = decltype(B)::value, c = decltype(C)::value;
            const bool constrained = (a == 0 && dx0) || (a == 2 && dx2) || (b == 0 && dy0) || (b == 2 && dy2) ||
                                     (c == 0 && dz0) || (c == 2 && dz2);
            const bool shared_hi = (a == 2 && sx2) || (b == 2 && sy2) || (c == 2 && sz2);
            const bool shared = shared_hi || (a == 0 && sx0) || (b == 0 && sy0) || (c == 0 && sz0);
            f(a, b, c, l0 + a + R * b + P * c, g0 + a + sy * b + sz * c, constrained,
              (shared ? 1 : 0) | (shared_hi ? 2 : 0));
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        // A brick with neighbours on all six sides and no Dirichlet face:
        // nothing is constrained, a low node is shared exactly on the
        // brick's low faces and every high node is shared.  Such bricks take
        // a copy of the visits with these flags folded in (a uniform branch;
        // 26.1 -> 25.6 us for the FP64 apply kernel at 64^3).
        auto inode = [&](auto A, auto B, auto C) {
            constexpr int a = decltype(A)::value, b = decltype(B)::value, c = decltype(C)::value;
            constexpr bool hi = a == 2 || b == 2 || c == 2;
            const bool shared = hi || (a == 0 && tx == 0) || (b == 0 && ty == 0) || (c == 0 && tz == 0);
            f(a, b, c, l0 + a + R * b + P * c, g0 + a + sy * b + sz * c, false, (shared ? 1 : 0) | (hi ? 2 : 0));
        };
        if (inner(m)) {
            inode(I0{}, I0{}, I0{}); inode(I1{}, I0{}, I0{}); inode(I0{}, I1{}, I0{}); inode(I1{}, I1{}, I0{});
            inode(I0{}, I0{}, I1{}); inode(I1{}, I0{}, I1{}); inode(I0{}, I1{}, I1{}); inode(I1{}, I1{}, I1{});
            if (lastx) { inode(I2{}, I0{}, I0{}); inode(I2{}, I1{}, I0{}); inode(I2{}, I0{}, I1{}); inode(I2{}, I1{}, I1{}); }
            if (lasty) { inode(I0{}, I2{}, I0{}); inode(I1{}, I2{}, I0{}); inode(I0{}, I2{}, I1{}); inode(I1{}, I2{}, I1{}); }
            if (lastz) { inode(I0{}, I0{}, I2{}); inode(I1{}, I0{}, I2{}); inode(I0{}, I1{}, I2{}); inode(I1{}, I1{}, I2{}); }
            if (lastx && lasty) { inode(I2{}, I2{}, I0{}); inode(I2{}, I2{}, I1{}); }
            if (lastx && lastz) { inode(I2{}, I0{}, I2{}); inode(I2{}, I1{}, I2{}); }
            if (lasty && lastz) { inode(I0{}, I2{}, I2{}); inode(I1{}, I2{}, I2{}); }
            if (lastx && lasty && lastz) inode(I2{}, I2{}, I2{});
            return;
        }
        node(I0{}, I0{}, I0{}); node(I1{}, I0{}, I0{}); node(I0{}, I1{}, I0{}); node(I1{}, I1{}, I0{});
        node(I0{}, I0{}, I1{}); node(I1{}, I0{}, I1{}); node(I0{}, I1{}, I1{}); node(I1{}, I1{}, I1{});
        if (lastx) { node(I2{}, I0{}, I0{}); node(I2{}, I1{}, I0{}); node(I2{}, I0{}, I1{}); node(I2{}, I1{}, I1{}); }
        if (lasty) { node(I0{}, I2{}, I0{}); node(I1{}, I2{}, I0{}); node(I0{}, I2{}, I1{}); node(I1{}, I2{}, I1{}); }
        if (lastz) { node(I0{}, I0{}, I2{}); node(I1{}, I0{}, I2{}); node(I0{}, I1{}, I2{}); node(I1{}, I1{}, I2{}); }
        if (lastx && lasty) { node(I2{}, I2{}, I0{}); node(I2{}, I2{}, I1{}); }
        if (lastx && lastz) { node(I2{}, I0{}, I2{}); node(I2{}, I1{}, I2{}); }
        if (lasty && lastz) { node(I0{}, I2{}, I2{}); node(I1{}, I2{}, I2{}); }
        if (lastx && lasty && lastz) node(I2{}, I2{}, I2{});
    }


    // Nodal fields are read through buffer resources based at the brick's
    // first node (uniform over the workgroup): node (2tx + a, 2ty + b,
    // 2tz + c) of the thread's cell lies at byte offset vo + a sizeof(T)
    // (per thread, immediate) plus b sy + c sz (uniform), so the loads need
    // no per-node 64-bit address arithmetic.  The brick's nodes span less
    // than 2^32 bytes from its first node; the records limit is the rest of
    // the array.  nodal_rsrc is the resource, nodal_vo the per-thread offset.
    template <typename T>
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t nodal_rsrc(const KMesh &m, const T *g) const
    {
        static_assert(sizeof(T) == 8 || sizeof(T) == 4, "FP64 or FP32 nodal arrays");
        const int64_t o = node_index(m, 2 * c0x, 2 * c0y, 2 * c0z);
        const int64_t rem = ((int64_t)m.NX * m.NY * m.NZ - o) * (int64_t)sizeof(T);
        const int nrec = (int)(unsigned)(rem > 0xFFFFFFFFll ? 0xFFFFFFFFll : rem);
        constexpr int kFormat = 0x00020000; // buffer descriptor word 3 for the gfx9 family
        return __builtin_amdgcn_make_buffer_rsrc((void *)(g + o), 0, nrec, kFormat);
    }
    template <typename T> __device__ __forceinline__ unsigned nodal_vo(const KMesh &m) const
    {
        return (unsigned)sizeof(T) * (unsigned)(2 * tx + m.NX * (2 * ty + m.NY * 2 * tz));
    }
    template <typename T>
    static __device__ __forceinline__ T nodal_load(__amdgpu_buffer_rsrc_t r, unsigned vofs, unsigned sofs)
    {
        if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, vofs, sofs, 0));
        else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, vofs, sofs, 0));
    }

    // Staging reads all 27 nodes of the thread's cell (of the brick's first
    // cell for a thread without one) and writes them to LDS.  A node that
    // several cells of the brick share is written by each of them with the
    // same value, so the staging needs no ownership test and no branches;
    // every read lies inside the mesh.
    template <typename T> __device__ __forceinline__ unsigned stage_vo(const KMesh &m) const
    {
        return valid ? nodal_vo<T>(m) : 0u;
    }
    template <typename T> __device__ __forceinline__ int stage_l0() const
    {
        return valid ? lds_index<T>(2 * tx, 2 * ty, 2 * tz) : 0;
    }

    // Stage a nodal field into LDS; Dirichlet nodes read as zero if mask.
    template <typename T>
    __device__ __forceinline__ void load(const KMesh &m, const T *__restrict__ g, T *lds, bool mask) const
    {
        const __amdgpu_buffer_rsrc_t r = nodal_rsrc(m, g);
        const unsigned vo = stage_vo<T>(m), sy = (unsigned)sizeof(T) * (unsigned)m.NX, sz = sy * (unsigned)m.NY;
        const int l0 = stage_l0<T>();
        constexpr int R = lds_row<T>(), P = lds_plane<T>();
        const unsigned f6 = mask ? m.dirichlet : 0u;
        const int gx0 = 2 * (c0x + (valid ? tx : 0)), gy0 = 2 * (c0y + (valid ? ty : 0)),
                  gz0 = 2 * (c0z + (valid ? tz : 0));
        const bool dx0 = (f6 & 1u) && gx0 == 0, dx2 = (f6 & 2u) && gx0 + 2 == m.NX - 1;
        const bool dy0 = (f6 & 4u) && gy0 == 0, dy2 = (f6 & 8u) && gy0 + 2 == m.NY - 1;
        const bool dz0 = (f6 & 16u) && gz0 == 0, dz2 = (f6 & 32u) && gz0 + 2 == m.NZ - 1;
        T v[27];
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    v[a + 3 * b + 9 * c] = nodal_load<T>(r, vo + (unsigned)(a * sizeof(T)), b * sy + c * sz);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const bool k = (a == 0 && dx0) || (a == 2 && dx2) || (b == 0 && dy0) || (b == 2 && dy2) ||
                                   (c == 0 && dz0) || (c == 2 && dz2);
                    lds[l0 + a + R * b + P * c] = k ? T(0) : v[a + 3 * b + 9 * c];
                }
    }

    // Node-parallel staging over a workgroup of WG threads (tid = the
    // thread's index in it) of NF fields of 8-byte entries: field f is read
    // from src[f] into the LDS region dst[f]; with MASK, a field with bit f
    // of maskbits set reads its Dirichlet nodes as zero.  Thread tid takes
    // the node column l_x = tid mod 9 of the rows (l_y, l_z) = row0 + RPI k,
    // row0 = tid div 9 and RPI = WG div 9 rows per step (the WG mod 9 threads
    // left over idle), so each step reads RPI whole 9-node rows, contiguous
    // along x, and the row index advances by constant steps (no per-node
    // division or multiply).  Every brick node is read once; all reads are
    // issued before the first LDS write.  Nodes beyond a clipped brick's valid
    // range are staged too: their reads stay inside the array or fall beyond
    // the buffer resource's range and read as zero, and no valid cell reads
    // their LDS slots.  Steps past the last row write to the row padding
    // (slot 9 of row 0), which nothing reads.
    template <int WG, int NF, bool MASK, typename T>
    __device__ __forceinline__ void stage_rows(const KMesh &m, int tid, const T *const (&src)[NF],
                                               T *const (&dst)[NF], unsigned maskbits) const
    {
        static_assert(sizeof(T) == 8, "8-byte entries (padded LDS rows)");
        constexpr int R = lds_row<T>(), P = lds_plane<T>();
        static_assert(R > BP, "the padding slot of row 0 takes the writes of the idle steps");
        constexpr int RPI = WG / BP, K = (BP * PZ + RPI - 1) / RPI;
        constexpr int DLY = RPI % BP, DLZ = RPI / BP;
        __amdgpu_buffer_rsrc_t rs[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) rs[f] = nodal_rsrc(m, src[f]);
        const unsigned NX = m.NX, NXY = (unsigned)m.NX * m.NY;
        asm volatile("" : "+v"(tid)); // set up per call: nothing kept live across stagings
        const int lx = tid % BP, row0 = tid / BP;
        const bool active = tid < RPI * BP;
        int ly = row0 % BP, lz = row0 / BP;
        unsigned vofs = 8u * ((unsigned)lx + NX * (unsigned)ly + NXY * (unsigned)lz);
        int lo = lx + R * ly + P * lz;
        const unsigned vstep = 8u * (DLY * NX + DLZ * NXY), vcarry = 8u * (NXY - BP * NX);
        T v[K][NF];
        int slot[K];
        bool con[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (k > 0) {
                ly += DLY;
                lz += DLZ;
                vofs += vstep;
                lo += DLY * R + DLZ * P;
                if (ly >= BP) {
                    ly -= BP;
                    lz += 1;
                    vofs += vcarry;
                    lo += P - BP * R;
                }
            }
            const bool ok = active && lz < PZ;
            slot[k] = ok ? lo : BP; // padding slot of row 0
            con[k] = MASK && ok && node_constrained(m, 2 * c0x + lx, 2 * c0y + ly, 2 * c0z + lz);
#pragma unroll
            for (int f = 0; f < NF; ++f) v[k][f] = nodal_load<T>(rs[f], ok ? vofs : 0u, 0);
        }
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int f = 0; f < NF; ++f) dst[f][slot[k]] = (MASK && ((maskbits >> f) & 1u) && con[k]) ? T(0) : v[k][f];
    }

    // The brick's NF (1 or 2) unmasked 8-byte fields, staged by its NT lanes.
    template <int NF, typename T>
    __device__ __forceinline__ void stage_nodes(const KMesh &m, const T *__restrict__ g0, T *l0s,
                                                const T *__restrict__ g1, T *l1s) const
    {
        if constexpr (NF == 1) {
            const T *src[1] = {g0};
            T *const dst[1] = {l0s};
            stage_rows<NT, 1, false, T>(m, t, src, dst, 0u);
        } else {
            const T *src[2] = {g0, g1};
            T *const dst[2] = {l0s, l1s};
            stage_rows<NT, 2, false, T>(m, t, src, dst, 0u);
        }
    }

    // NF FP64 fields by the brick's lanes (the slabs' interface).
    template <int NF>
    __device__ __forceinline__ void stage(const KMesh &m, const double *const (&src)[NF], double *const (&dst)[NF]) const
    {
        stage_rows<NT, NF, false, double>(m, t, src, dst, 0u);
    }

    // NF FP64 fields over a workgroup of WG threads; bit f of maskbits: field f
    // reads its Dirichlet nodes as zero.
    template <int WG, int NF>
    __device__ __forceinline__ void stage_nodes_wg(const KMesh &m, int tid, const double *const (&src)[NF],
                                                   double *const (&dst)[NF], unsigned maskbits) const
    {
        if (maskbits) stage_rows<WG, NF, true, double>(m, tid, src, dst, maskbits);
        else stage_rows<WG, NF, false, double>(m, tid, src, dst, 0u);
    }

    // The cell's 27 nodal values with its Dirichlet nodes read as zero (the
    // constrained columns are removed); bricks away from Dirichlet faces
    // skip the test (uniform branch).
    template <typename T> __device__ __forceinline__ void gather27_dirichlet(const KMesh &m, const T *lds, T *v) const
    {
        gather27(lds, v);
        if (!touches_dirichlet(m)) return;
        const unsigned f6 = m.dirichlet;
        const int gx0 = 2 * (c0x + tx), gy0 = 2 * (c0y + ty), gz0 = 2 * (c0z + tz);
        const bool dx0 = (f6 & 1u) && gx0 == 0, dx2 = (f6 & 2u) && gx0 + 2 == m.NX - 1;
        const bool dy0 = (f6 & 4u) && gy0 == 0, dy2 = (f6 & 8u) && gy0 + 2 == m.NY - 1;
        const bool dz0 = (f6 & 16u) && gz0 == 0, dz2 = (f6 & 32u) && gz0 + 2 == m.NZ - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const bool k = (a == 0 && dx0) || (a == 2 && dx2) || (b == 0 && dy0) || (b == 2 && dy2) ||
                                   (c == 0 && dz0) || (c == 2 && dz2);
                    v[a + 3 * b + 9 * c] = k ? T(0) : v[a + 3 * b + 9 * c];
                }
    }

    // The cell's 27 nodal values from LDS (zero for threads without a cell).
    template <typename T> __device__ __forceinline__ void gather27(const T *lds, T *v) const
    {
        const int l0 = valid ? lds_index<T>(2 * tx, 2 * ty, 2 * tz) : 0;
        constexpr int R = lds_row<T>(), P = lds_plane<T>();
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a) v[a + 3 * b + 9 * c] = lds[l0 + a + R * b + P * c];
    }

    // Cell results, node-major: E[local * NT + thread].  A thread without a
    // cell stores whatever it computed: node_sum reads only the lower
    // neighbours of a valid cell within the brick, and those are valid too.
    template <typename T> __device__ __forceinline__ void store_cell(T *E, const T *v) const
    {
#pragma unroll
        for (int i = 0; i < 27; ++i) E[i * NT + t] = v[i];
    }

    // Lane shift within the 16-lane rows of the wavefront (DPP row_shr:S):
    // lane i takes lane i - S of its row, the first S lanes of a row take 0.
    template <int S, typename T> static __device__ __forceinline__ T row_shr(T v)
    {
        static_assert(S >= 1 && S <= 15, "row shift");
        constexpr int ctrl = 0x110 + S;
        if constexpr (sizeof(T) == 8) {
            const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
            const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, ctrl, 0xF, 0xF, true);
            const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), ctrl, 0xF, 0xF, true);
            return __builtin_bit_cast(T, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
        } else {
            return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xF, 0xF, true));
        }
    }

    // Node sums in registers.  On entry u holds this cell's 27 contributions;
    // on exit u[a + 3b + 9c] is the sum over the brick's cells containing
    // that node for every node the cell owns (the entries of index 2 of a
    // cell that is not the last in that direction are partial).  Cells are
    // lanes t = tx + 4 ty + 16 tz, so the low neighbour in x is lane t - 1
    // and in y lane t - 4, both in the same 16-lane row (a DPP row shift;
    // the first cell of an x line is masked, the first of a y line is at a
    // row's start and takes zero), and in z lane t - 16, exchanged through
    // LDS (xch, 9 NT values).  The sums run x, then y, then z: a fixed order.
    // All lanes of the wavefront must call it.
    template <typename T> __device__ __forceinline__ void assemble27(T *u, T *xch) const
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) { // x: (b, c) = (i % 3, i / 3)
            const T nb = row_shr<1>(u[2 + 3 * i]);
            u[3 * i] += tx > 0 ? nb : T(0);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < 3; ++a) u[a + 9 * c] += row_shr<4>(u[a + 6 + 9 * c]);
#pragma unroll
        for (int i = 0; i < 9; ++i) xch[i * NT + t] = u[18 + i];
        __syncthreads();
        const int src = tz > 0 ? t - BB * BB : t;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const T nb = xch[i * NT + src];
            u[i] += tz > 0 ? nb : T(0);
        }
    }

    // Sum over the brick's cells containing local node (a, b, c) of this
    // thread's cell: the cell itself and, for index 0 in a direction, the
    // neighbour on the low side (local index 2 there).  Branch free: a
    // missing neighbour (brick edge) reads this cell's slot, weighted by 0.
    template <typename T> __device__ __forceinline__ T node_sum(const T *E, int a, int b, int c) const
    {
        T s = E[(a + 3 * b + 9 * c) * NT + t];
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                for (int dx = 0; dx < 2; ++dx) {
                    if (dx + dy + dz == 0) continue;
                    if ((dx && a != 0) || (dy && b != 0) || (dz && c != 0)) continue;
                    const bool ok = !((dx && tx == 0) || (dy && ty == 0) || (dz && tz == 0));
                    const int loc = (a + 2 * dx) + 3 * (b + 2 * dy) + 9 * (c + 2 * dz);
                    const int nb = ok ? t - dx - BB * dy - BB * BB * dz : t;
                    s += (ok ? T(1) : T(0)) * E[loc * NT + nb];
                }
        return s;
    }
};

// ---------------------------------------------------------------------------
// Shared-node combine.  The nodes that several bricks touch lie on the
// internal brick planes of some direction.  A node's value is the sum of the
// face partials of the 2, 4 or 8 bricks containing it, in a fixed order (z
// outer, then y, then x; lower brick first).  Shared Dirichlet nodes: DMODE 1
// writes y = x (identity rows of an operator), DMODE 2 writes y = 1 (its
// diagonal), DMODE 3 writes 0 (a right-hand side), DMODE 0 sums them like
// every other node (a plain nodal field such as a gradient).  DMODE 4 is
// DMODE 2 with the reciprocal of every other sum stored (the inverse
// diagonal).
// ---------------------------------------------------------------------------

// Brick-owned combine: a wavefront per brick (numbered like the brick
// kernels, XCD-contiguously), two per slab of two or four sub-bricks.  Each shared node is finished
// by the one brick that holds it at local index 0 in every direction in
// which it is shared: the brick's nodes on its low faces that lie on
// internal brick planes, without its shared high faces (the next brick's
// low faces).  For a 4x4x4 brick with lower neighbours in x, y and z that is
// up to 64 + 56 + 49 nodes (217 for a brick at the far end of the mesh in
// every direction), at most four per lane; a slab has up to 297 + 264 + 64 =
// 625 over two wavefronts, five per lane.  They are
// enumerated in three slabs: l_z = 0 (runs along x); l_y = 0 (runs along x);
// l_x = 0 (runs along y, where the x-face slots are contiguous).  The
// partials are summed in the fixed order above (the same order as a pass
// that enumerates the shared nodes flat, which this pass replaced with
// bitwise the same results); all loads of a lane's nodes are issued before
// the sums.
// The visit for one brick (or slab: BR gives the extents, CX x BB x BB cells,
// and the face-buffer slots); INNER: a brick with neighbours on all six sides
// and no Dirichlet face, for which the ranges, the sharing flags and the
// divisions are compile-time constants and nothing is constrained.  L lanes
// finish one brick.
template <typename T, bool SKIP_CONSTRAINED, int L, bool INNER, typename BR, typename F>
__device__ __forceinline__ void combine_brick_nodes(const KMesh &m, const BR &br, int nbx, int nby, int nbz,
                                                    int lane, const T *__restrict__ face, F f)
{
    constexpr int BX = BR::CX;
    // lower neighbour: the low face is shared
    const bool fx = INNER || br.bx > 0, fy = INNER || br.by > 0, fz = INNER || br.bz > 0;
    // local range without a shared high face
    const int ex = INNER ? 2 * BX : 2 * br.ncx + (br.bx == nbx - 1 ? 1 : 0);
    const int ey = INNER ? 2 * BB : 2 * br.ncy + (br.by == nby - 1 ? 1 : 0);
    const int ez = INNER ? 2 * BB : 2 * br.ncz + (br.bz == nbz - 1 ? 1 : 0);
    const int z0 = fz ? 1 : 0, y0 = fy ? 1 : 0;
    const int nzs = fz ? ex * ey : 0, nys = fy ? ex * (ez - z0) : 0, nxs = fx ? (ey - y0) * (ez - z0) : 0;
    const int tot = nzs + nys + nxs;
    // small exact divisions: floor((j + 1/2) / w) for j < 1024, w <= 33
    const float iex = 1.0f / (float)ex, iw = 1.0f / (float)(ey - y0);
    auto div = [&](int j, int w, float iw_) { return INNER ? j / w : (int)(((float)j + 0.5f) * iw_); };
    // nodes per lane: a z, a y and an x face at most over the brick's lanes
    constexpr int K = ((2 * BX + 1) * BP + (2 * BX + 1) * 2 * BB + 2 * BB * 2 * BB + L - 1) / L;
    bool has[K], con[K];
    int64_t g[K];
    T v[K][8];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int j = lane + L * k;
        has[k] = j < tot;
        int lx = 0, ly = 0, lz = 0;
        if (j < nzs) {
            ly = div(j, ex, iex);
            lx = j - ly * ex;
        } else if ((j -= nzs) < nys) {
            const int q = div(j, ex, iex);
            lz = z0 + q;
            lx = j - q * ex;
        } else {
            j -= nys;
            const int w = ey - y0, q = div(j, w, iw);
            lz = z0 + q;
            ly = y0 + j - q * w;
        }
        if (!has[k]) lx = ly = lz = 0;
        const int gx = 2 * br.c0x + lx, gy = 2 * br.c0y + ly, gz = 2 * br.c0z + lz;
        con[k] = !INNER && has[k] && node_constrained(m, gx, gy, gz);
        g[k] = node_index(m, gx, gy, gz);
        const bool read = has[k] && !(SKIP_CONSTRAINED && con[k]);
        const bool sx = lx == 0 && fx, sy = ly == 0 && fy, sz = lz == 0 && fz;
        const int kx0 = sx ? br.bx - 1 : br.bx, lx0 = sx ? 2 * BX : lx;
        const int ky0 = sy ? br.by - 1 : br.by, ly0 = sy ? 2 * BB : ly;
        const int kz0 = sz ? br.bz - 1 : br.bz, lz0 = sz ? 2 * BB : lz;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int ex_ = e & 1, ey_ = (e >> 1) & 1, ez_ = e >> 2;
            v[k][e] = T(0);
            if (read && (!ex_ || sx) && (!ey_ || sy) && (!ez_ || sz)) {
                const int b = (kx0 + ex_) + nbx * ((ky0 + ey_) + nby * (kz0 + ez_));
                v[k][e] = face[(int64_t)b * BR::NFACE + BR::face_slot_of(ex_ ? 0 : lx0, ey_ ? 0 : ly0, ez_ ? 0 : lz0)];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (!has[k]) continue;
        T s = v[k][0];
#pragma unroll
        for (int e = 1; e < 8; ++e) s += v[k][e];
        f(g[k], con[k], (SKIP_CONSTRAINED && con[k]) ? T(0) : s);
    }
}

template <typename T, bool SKIP_CONSTRAINED, typename F>
__device__ __forceinline__ void combine_brick_visit(const KMesh &m, int brick, int lane, const T *__restrict__ face,
                                                    F f)
{
    const Brick br(m, lane, brick);
    const int nbx = (m.nx + BB - 1) / BB, nby = (m.ny + BB - 1) / BB, nbz = (m.nz + BB - 1) / BB;
    constexpr int L = BNT; // a wavefront per brick
    if (br.inner(m)) combine_brick_nodes<T, SKIP_CONSTRAINED, L, true>(m, br, nbx, nby, nbz, lane, face, f);
    else combine_brick_nodes<T, SKIP_CONSTRAINED, L, false>(m, br, nbx, nby, nbz, lane, face, f);
}

// ---------------------------------------------------------------------------
// Slabs.  A workgroup of W wavefronts owns 4W x 4 x 4 cells, W 4x4x4
// sub-bricks side by side along x, one per wavefront, over (8W + 1) x 9 x 9
// nodes staged once in LDS.  The cells are computed as in a brick; what
// changes is how the nodes travel: staged and finished row by row by the
// whole workgroup, the node sums passing through LDS, with a few bit tests
// per row where a brick visits its owned nodes cell by cell, 27 divergent
// groups (a wavefront alone on its CU spent 4200 of its 13700 cycles there,
// 7000 on a brick at the boundary of the mesh).
// W = 4: a brick's rows are 9 nodes, 72 or 36 bytes of a 128-byte line; on
// 128^3 cells in FP32 the brick kernel made 9.7M L2 reads and 8.4M L2 writes
// for 1.7M lines and kept the address units busy 79 % of the time, and a
// workgroup waited 33000 of its 48000 cycles for its staging reads (11800 of
// 25500 now).  A slab's rows are 33 nodes; it shares three quarters of the
// nodes that four bricks share with their neighbours, and a quarter of those
// on planes across x, which the combine pass can only write one by one.
// W = 1 spreads a small mesh over four times the CUs; W = 2 is between them.
// ---------------------------------------------------------------------------

// A visitor whose arrays must stay in registers has to be inlined.
#define MF_INLINE __attribute__((always_inline))

// f(0), f(1), ... with the index a compile-time constant (a loop over an
// array in registers that the optimizer might split instead of unrolling).
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

__host__ __device__ inline unsigned ceil_div(int n, int d) { return (unsigned)(n + d - 1) / (unsigned)d; }
template <int W> __host__ __device__ inline int64_t n_slabs(const KMesh &m)
{
    return (int64_t)ceil_div(m.nx, W * BB) * ceil_div(m.ny, BB) * ceil_div(m.nz, BB);
}

// LDS of W > 1 beside the staged fields: the sums on the sub-bricks' x-high
// faces (81 each; read in whole steps of rows, hence the padding).
template <int W> __host__ __device__ constexpr int slab_xhi() { return W > 1 ? 81 * (W - 1) + 8 : 0; }

template <int W_, int R_ = (W_ == 1 ? 10 : 8 * W_ + 4)> struct Slab {
    static constexpr int W = W_, NT = W * BNT;
    static constexpr int RX = 2 * W * BB, SP = RX + 1; // nodes along x without and with the high face
    static constexpr int CX = W * BB;
    // Face buffer: one slot per node, surface nodes used; the x-low face, the
    // x-high face, then the rows without their ends, so that a combine pass
    // reads the x faces contiguously too (with whole rows of 9 the 49 nodes of
    // a brick's x face lay on as many lines: convective apply on 56^3 cells 38.5
    // us, 36.1 so; plain FP64 on 77^3 53.4, 50.6).
    static constexpr int NFACE = SP * BP * BP, ROWS = BP * BP;
    static __device__ __forceinline__ constexpr int face_row(int lx) // slots from one row (ly + 9 lz) to the next
    {
        return lx == 0 || lx == SP - 1 ? 1 : SP - 2;
    }
    static __device__ __forceinline__ constexpr int face_slot_of(int lx, int ly, int lz)
    {
        const int start = lx == 0 ? 0 : lx == SP - 1 ? ROWS : 2 * ROWS + lx - 1;
        return start + face_row(lx) * (ly + BP * lz);
    }
    // LDS layout of a staged field: node (lx, ly, lz) at lx + R ly + plane lz.
    // A wavefront gathers nodes (2tx + a, 2ty + b, 2tz + c): with R = 4 (mod
    // 16) the 16 lanes of a z plane fall on 16 different 8-byte banks; the
    // FP32 planes are padded so that two z planes of lanes do not meet.  W = 1
    // keeps rows of 10: with 12 three staged fields would leave six
    // workgroups per CU instead of eight.
    static constexpr int R = R_;
    static_assert(R >= SP, "a padding slot in row 0 takes the writes of idle threads");
    template <typename T> static __host__ __device__ constexpr int plane()
    {
        return sizeof(T) == 8 ? R * BP : (R * BP + 15) / 32 * 32 + 16;
    }
    template <typename T> static __host__ __device__ constexpr int field() { return plane<T>() * BP; }

    int brick;         // natural slab index (x fastest)
    int bx, by, bz;    // slab coordinates
    int c0x, c0y, c0z; // first cell
    int ncx, ncy, ncz; // valid cells per direction
    int tid, w, t;     // thread, wavefront (uniform), lane
    int tx, ty, tz;    // cell within the wavefront's sub-brick
    bool valid;

    __device__ __forceinline__ Slab(const KMesh &m, int tid_) : Slab(m, tid_, Brick::xcd_index()) {}
    __device__ __forceinline__ Slab(const KMesh &m, int tid_, int b) : brick(b), tid(tid_)
    {
        const int nbx = (int)ceil_div(m.nx, CX), nby = (int)ceil_div(m.ny, BB);
        const int q = (int)udiv((unsigned)brick, (unsigned)nbx, W == 1 ? m.rbx : W == 2 ? m.rs2 : m.rs4);
        bx = brick - q * nbx;
        bz = (int)udiv((unsigned)q, (unsigned)nby, m.rby);
        by = q - bz * nby;
        place(m, CX, BB);
    }
    // Cells and lanes of slab (bx, by, bz), slabs sx and s cells apart.
    __device__ __forceinline__ void place(const KMesh &m, int sx, int s)
    {
        c0x = bx * sx;
        c0y = by * s;
        c0z = bz * s;
        ncx = min(CX, m.nx - c0x);
        ncy = min(BB, m.ny - c0y);
        ncz = min(BB, m.nz - c0z);
        w = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / BNT);
        t = tid % BNT;
        tx = t & (BB - 1);
        ty = (t / BB) & (BB - 1);
        tz = t / (BB * BB);
        valid = w * BB + tx < ncx && ty < ncy && tz < ncz;
    }
    // (for Tile, which sets the slab coordinates itself)
    __device__ __forceinline__ Slab(int b, int tid_) : brick(b), tid(tid_) {}
    __device__ __forceinline__ int64_t cell_index(const KMesh &m) const
    {
        return (int64_t)(c0x + w * BB + tx) + (int64_t)m.nx * ((c0y + ty) + (int64_t)m.ny * (c0z + tz));
    }
    // The slab's faces as bits (x low, x high, y low, ...): those shared with
    // a neighbouring slab, and those on a Dirichlet face of the mesh.
    __device__ __forceinline__ unsigned shared_faces(const KMesh &m) const
    {
        return (bx > 0 ? 1u : 0u) | (c0x + CX < m.nx ? 2u : 0u) | (by > 0 ? 4u : 0u) | (c0y + BB < m.ny ? 8u : 0u) |
               (bz > 0 ? 16u : 0u) | (c0z + BB < m.nz ? 32u : 0u);
    }
    __device__ __forceinline__ unsigned dirichlet_faces(const KMesh &m) const { return m.dirichlet & ~shared_faces(m); }
    // Neighbours on all six sides (and so no Dirichlet face).
    __device__ __forceinline__ bool inner(const KMesh &m) const { return shared_faces(m) == 63u; }
    // The faces on which local node (lx, ly, lz) lies.
    __device__ __forceinline__ unsigned x_faces(int lx) const { return (lx == 0 ? 1u : 0u) | (lx == 2 * ncx ? 2u : 0u); }
    __device__ __forceinline__ unsigned yz_faces(int ly, int lz) const
    {
        return (ly == 0 ? 4u : 0u) | (ly == 2 * ncy ? 8u : 0u) | (lz == 0 ? 16u : 0u) | (lz == 2 * ncz ? 32u : 0u);
    }

    // Visit the slab's nodes with lx < 8W, eight rows per step: thread tid takes
    // node lx = tid mod 8W of the rows r0 + 8 k, r0 = tid / 8W, row = ly + 9 lz.
    // Since a plane has one row more than a step, ly = r0 - k (+ 9) and
    // lz = k (- 1): everything is a constant step per k and one comparison,
    // and the rows on a slab face are known per step (see the finishing
    // pass).  f(k, slot, off, ly, lz, ok) with k a constant, slot the node in a
    // staged field of T, off its element offset from the slab's first node in
    // a nodal array; ok is false only beyond the last row (last step).
    static constexpr int RPS = NT / RX, STEPS = (BP * BP + RPS - 1) / RPS;
    static_assert(RPS == BP - 1 && STEPS == 11, "the row arithmetic of for_rows");
    template <typename T, typename F> __device__ __forceinline__ void for_rows(const KMesh &m, F f) const
    {
        int i = tid;
        asm volatile("" : "+v"(i)); // set up per call: nothing kept live across visits
        const int lx = i % RX, r0 = i / RX;
        constexpr int P = plane<T>();
        const int slot0 = lx + R * r0;
        const unsigned off0 = (unsigned)lx + (unsigned)m.NX * (unsigned)r0;
        const unsigned S = (unsigned)m.NX * ((unsigned)m.NY - 1u), C = (unsigned)m.NX * (BP - (unsigned)m.NY);
        static_for<STEPS>([&](auto kc) MF_INLINE {
            constexpr int k = decltype(kc)::value;
            if constexpr (k < STEPS - 1) {
                const bool lo = r0 < k; // the row lies in plane k - 1
                f(kc, slot0 + (P - R) * k + (lo ? R * BP - P : 0), off0 + k * S + (lo ? C : 0u), r0 - k + (lo ? BP : 0),
                  k - (lo ? 1 : 0), true);
            } else { // row 80 (thread row 0), the last one
                f(kc, lx + R * (BP - 1) + P * (BP - 1), (unsigned)lx + (unsigned)m.NX * ((BP - 1) + (unsigned)m.NY * (BP - 1)),
                  BP - 1, BP - 1, r0 == 0);
            }
        });
    }
    // The same for the nodes lx = 8W: 81 of them, f(k, ...) for row tid + NT k.
    static constexpr int ESTEPS = (BP * BP + NT - 1) / NT;
    template <typename T, typename F> __device__ __forceinline__ void for_edge(const KMesh &m, F f) const
    {
        int i = tid;
        asm volatile("" : "+v"(i));
        static_for<ESTEPS>([&](auto kc) MF_INLINE {
            constexpr int k = decltype(kc)::value;
            const int row = i + NT * k, lz = row / BP, ly = row - lz * BP;
            f(kc, RX + R * ly + plane<T>() * lz, (unsigned)RX + (unsigned)m.NX * ((unsigned)ly + (unsigned)m.NY * lz), ly,
              lz, row < BP * BP);
        });
    }
    static constexpr int NV = STEPS + ESTEPS; // visited nodes per thread

    // Stage NF nodal fields; every read is issued before the first LDS write.
    // Rows are read from the slab's first node through a buffer resource (as
    // Brick::stage_rows): reads beyond a clipped slab stay inside the array
    // or past its end, where they return zero, and no valid cell uses them.
    template <int NF, typename T>
    __device__ __forceinline__ void stage(const KMesh &m, const T *const (&src)[NF], T *const (&dst)[NF]) const
    {
        __amdgpu_buffer_rsrc_t rs[NF];
        const int64_t o = node_index(m, 2 * c0x, 2 * c0y, 2 * c0z);
        const int64_t rem = ((int64_t)m.NX * m.NY * m.NZ - o) * (int64_t)sizeof(T);
        const int nrec = (int)(unsigned)(rem > 0xFFFFFFFFll ? 0xFFFFFFFFll : rem);
#pragma unroll
        for (int f = 0; f < NF; ++f) rs[f] = __builtin_amdgcn_make_buffer_rsrc((void *)(src[f] + o), 0, nrec, 0x00020000);
        T v[NV][NF];
        int at[NV];
        auto node = [&](int k, int slot, unsigned off, bool ok) MF_INLINE {
            at[k] = ok ? slot : SP; // idle threads write to the padding slot of row 0
            const unsigned vofs = ok ? (unsigned)sizeof(T) * off : 0u;
#pragma unroll
            for (int f = 0; f < NF; ++f) v[k][f] = Brick::nodal_load<T>(rs[f], vofs, 0);
        };
        for_rows<T>(m, [&](auto k, int slot, unsigned off, int, int, bool ok) MF_INLINE { node(k, slot, off, ok); });
        for_edge<T>(m, [&](auto k, int slot, unsigned off, int, int, bool ok) MF_INLINE { node(STEPS + k, slot, off, ok); });
#pragma unroll
        for (int k = 0; k < NV; ++k)
#pragma unroll
            for (int f = 0; f < NF; ++f) dst[f][at[k]] = v[k][f];
    }

    // Stage as above with the first field formed on the way, p = z + beta p_old
    // from src[0] = z and src[1] = p_old (dst[0] takes p, dst[f] src[f + 1]):
    // the direction update of a CG iteration, with the previous iteration's
    // x += alpha p_old.  p also goes to pn.  x and pn: each node from the one
    // slab that owns it.  mid(alpha, beta) runs once all reads are issued; where
    // it returns false (in every thread alike), only x is updated and false
    // is returned.
    template <int NF, typename T, typename M>
    __device__ __forceinline__ bool stage_direction(const KMesh &m, const T *const (&src)[NF], T *const (&dst)[NF - 1],
                                                    T *__restrict__ pn, T *__restrict__ x, M mid) const
    {
        __amdgpu_buffer_rsrc_t rs[NF + 1];
        const int64_t o = node_index(m, 2 * c0x, 2 * c0y, 2 * c0z);
        const int64_t rem = ((int64_t)m.NX * m.NY * m.NZ - o) * (int64_t)sizeof(T);
        const int nrec = (int)(unsigned)(rem > 0xFFFFFFFFll ? 0xFFFFFFFFll : rem);
#pragma unroll
        for (int f = 0; f <= NF; ++f)
            rs[f] = __builtin_amdgcn_make_buffer_rsrc((void *)((f < NF ? src[f] : x) + o), 0, nrec, 0x00020000);
        const int ox = owned_end(m.nx, c0x, CX), oy = owned_end(m.ny, c0y, BB), oz = owned_end(m.nz, c0z, BB);
        const int lx = tid % RX;
        T v[NV][NF + 1];
        auto read = [&](int k, unsigned off, bool okx, int ly, int lz, bool ok) MF_INLINE {
            const unsigned vofs = ok ? (unsigned)sizeof(T) * off : 0u;
#pragma unroll
            for (int f = 0; f < NF; ++f) v[k][f] = Brick::nodal_load<T>(rs[f], vofs, 0);
            v[k][NF] = Brick::nodal_load<T>(rs[NF], okx && ly <= oy && lz <= oz ? vofs : 0u, 0);
        };
        for_rows<T>(m, [&](auto k, int, unsigned off, int ly, int lz, bool ok) MF_INLINE {
            read(k, off, lx <= ox, ly, lz, ok);
        });
        for_edge<T>(m, [&](auto k, int, unsigned off, int ly, int lz, bool ok) MF_INLINE {
            read(STEPS + k, off, RX <= ox, ly, lz, ok);
        });
        T alpha, beta;
        const bool go = mid(alpha, beta);
        T *const pb = pn + o, *const xb = x + o;
        auto put = [&](int k, int slot, unsigned off, bool okx, int ly, int lz, bool ok) MF_INLINE {
            const bool own = ok && okx && ly <= oy && lz <= oz;
            if (own) xb[off] = v[k][NF] + alpha * v[k][1];
            if (!go) return;
            const T p = v[k][0] + beta * v[k][1];
            const int at = ok ? slot : SP; // as in stage
            dst[0][at] = p;
#pragma unroll
            for (int f = 2; f < NF; ++f) dst[f - 1][at] = v[k][f];
            if (own) pb[off] = p;
        };
        for_rows<T>(m, [&](auto k, int slot, unsigned off, int ly, int lz, bool ok) MF_INLINE {
            put(k, slot, off, lx <= ox, ly, lz, ok);
        });
        for_edge<T>(m, [&](auto k, int slot, unsigned off, int ly, int lz, bool ok) MF_INLINE {
            put(STEPS + k, slot, off, RX <= ox, ly, lz, ok);
        });
        return go;
    }
    // Last local node index that this slab, not the next one, owns along a
    // direction of n cells, with `size` cells per slab from cell c0 on.
    static __device__ __forceinline__ int owned_end(int n, int c0, int size)
    {
        return c0 + size < n ? 2 * size - 1 : 2 * (n - c0);
    }

    // The node sums at the visited nodes (from v[STEPS] on: the edge), all read
    // together: the node array, plus the left sub-brick's part on the planes
    // between sub-bricks (whose threads are the same in every step).
    template <typename T>
    __device__ __forceinline__ void node_values(const KMesh &m, const T *nod, const T *xhi, T (&v)[NV]) const
    {
        read_nodes(m, nod, v);
        if constexpr (W == 1) return;
        const int lx = tid % RX;
        if ((lx & 7) == 0 && lx > 0 && lx < 2 * ncx) {
            const T *h = xhi + 81 * ((lx >> 3) - 1) + tid / RX; // row = ly + 9 lz
            T s[STEPS];
#pragma unroll
            for (int k = 0; k < STEPS; ++k) s[k] = h[RPS * k]; // rows beyond the last one: padding
#pragma unroll
            for (int k = 0; k < STEPS; ++k) v[k] += s[k];
        }
    }
    // A staged field at the visited nodes.
    template <typename T> __device__ __forceinline__ void read_nodes(const KMesh &m, const T *f, T (&v)[NV]) const
    {
        for_rows<T>(m, [&](auto k, int slot, unsigned, int, int, bool) MF_INLINE { v[k] = f[slot]; });
        for_edge<T>(m, [&](auto k, int slot, unsigned, int, int, bool ok) MF_INLINE { v[STEPS + k] = f[ok ? slot : 0]; });
    }

    template <typename T> __device__ __forceinline__ int cell_slot() const
    {
        return valid ? 2 * (w * BB + tx) + R * 2 * ty + plane<T>() * 2 * tz : 0;
    }
    // The cell's 27 nodal values from LDS.
    template <typename T> __device__ __forceinline__ void gather27(const T *lds, T *v) const
    {
        const T *p = lds + cell_slot<T>();
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a) v[a + 3 * b + 9 * c] = p[a + R * b + plane<T>() * c];
    }
    // The same with the cell's Dirichlet nodes read as zero.
    template <typename T> __device__ __forceinline__ void gather27_dirichlet(const KMesh &m, const T *lds, T *v) const
    {
        gather27(lds, v);
        const unsigned f6 = dirichlet_faces(m);
        if (f6 == 0u) return;
        const int lx = 2 * (w * BB + tx);
        const unsigned lo = (x_faces(lx) | yz_faces(2 * ty, 2 * tz)) & f6;
        const unsigned hi = (x_faces(lx + 2) | yz_faces(2 * ty + 2, 2 * tz + 2)) & f6;
        const bool dx0 = lo & 1u, dx2 = hi & 2u, dy0 = lo & 4u, dy2 = hi & 8u, dz0 = lo & 16u, dz2 = hi & 32u;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const bool k = (a == 0 && dx0) || (a == 2 && dx2) || (b == 0 && dy0) || (b == 2 && dy2) ||
                                   (c == 0 && dz0) || (c == 2 && dz2);
                    v[a + 3 * b + 9 * c] = k ? T(0) : v[a + 3 * b + 9 * c];
                }
    }

    // Node sums of the wavefront's sub-brick (as Brick::assemble27, within
    // the wavefront) written to the node array nod (layout of a staged field).
    // xch: the wavefront's own 9 x 64 values (with W = 1 it may overlay nod:
    // it is read before the sums are written).  Every cell writes all its 27
    // entries, the ones of index 2 first: where another cell of the
    // sub-brick owns that node, its sum is written later by the same
    // wavefront and stays (LDS operations of a wavefront are executed in
    // order), so no write is masked.  Only the sub-brick's x-high face, which
    // the next sub-brick's wavefront writes, goes to xhi (81 values per
    // sub-brick but the last, added when the nodes are read).
    template <typename T> __device__ __forceinline__ void assemble(T *u, T *xch, T *nod, T *xhi) const
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const T nb = Brick::row_shr<1>(u[2 + 3 * i]);
            u[3 * i] += tx > 0 ? nb : T(0);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < 3; ++a) u[a + 9 * c] += Brick::row_shr<4>(u[a + 6 + 9 * c]);
#pragma unroll
        for (int i = 0; i < 9; ++i) xch[i * BNT + t] = u[18 + i];
        wave_lds_fence();
        const int src = tz > 0 ? t - BB * BB : t;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const T nb = xch[i * BNT + src];
            u[i] += tz > 0 ? nb : T(0);
        }
        if (!valid) return;
        // x-high face entries of the sub-brick's last cells: beside the node array
        const bool side = W > 1 && tx == BB - 1 && w * BB + BB < ncx;
        T *const p = nod + cell_slot<T>();
        T *const px = side ? xhi + 81 * w + 2 * ty + BP * 2 * tz : p + 2;
        const int sy = side ? 1 : R, sz = side ? BP : plane<T>();
#pragma unroll
        for (int c = 2; c >= 0; --c)
#pragma unroll
            for (int b = 2; b >= 0; --b) {
                px[sy * b + sz * c] = u[2 + 3 * b + 9 * c];
                wave_lds_order();
                p[1 + R * b + plane<T>() * c] = u[1 + 3 * b + 9 * c];
                p[R * b + plane<T>() * c] = u[3 * b + 9 * c];
                wave_lds_order();
            }
    }
    // LDS written by this wavefront is read by its other lanes.
    static __device__ __forceinline__ void wave_lds_fence()
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // Keeps the program order of LDS writes to the same address by different lanes.
    static __device__ __forceinline__ void wave_lds_order()
    {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    }
};

// Finish the nodes of a slab: v holds the node sums (node_values), xv the
// vector x at the nodes (only read on Dirichlet nodes, and for the energy).
// Complete nodes go to y, shared ones to the slab's face-buffer slots;
// Dirichlet rows get y_i = x_i.  With CG, energy gains x_i times the slab's
// partial sum, and x_i^2 for a Dirichlet node counted once, by the slab that
// finishes it.
template <typename T, bool CG, typename SL>
__device__ __forceinline__ void finish_nodes(const KMesh &m, const SL &br, T *__restrict__ y, T *__restrict__ face,
                                             T (&v)[SL::NV], T (&xv)[SL::NV], double &energy)
{
    constexpr int K = SL::STEPS;
    T *const yb = y + node_index(m, 2 * br.c0x, 2 * br.c0y, 2 * br.c0z);
    T *const fb = face + (int64_t)br.brick * SL::NFACE;
    const int lx = br.tid % SL::RX, r0 = br.tid / SL::RX, fstep = SL::RPS * SL::face_row(lx);
    T *const f0 = fb + SL::face_slot_of(lx, r0, 0), *const fe = fb + SL::face_slot_of(SL::RX, br.tid, 0); // row r: ly = r, lz = 0
    const unsigned shf = br.shared_faces(m), dirf = br.dirichlet_faces(m);
    if (shf == 63u) { // neighbours on all sides
        // steps 0, 9 and 10 are the two z faces; of step k in between the
        // rows r0 = k (ly = 0) and k - 1 (ly = 8) lie on the y faces
        br.template for_rows<T>(m, [&](auto kc, int, unsigned off, int, int, bool ok) MF_INLINE {
            constexpr int k = decltype(kc)::value;
            T *d = f0 + k * fstep;
            if constexpr (k >= 1 && k <= 8) d = (lx == 0 || r0 == k || r0 == k - 1) ? d : yb + off;
            if constexpr (CG) energy += ok ? (double)xv[k] * (double)v[k] : 0.0;
            if (k < K - 1 || ok) *d = v[k];
        });
        br.template for_edge<T>(m, [&](auto kc, int, unsigned, int, int, bool ok) MF_INLINE {
            constexpr int k = decltype(kc)::value;
            if constexpr (CG) energy += ok ? (double)xv[K + k] * (double)v[K + k] : 0.0;
            if (ok) fe[k * SL::NT] = v[K + k];
        });
        return;
    }
    // per node the faces it lies on, tested against the slab's shared and
    // Dirichlet faces (uniform masks)
    const int ex = 2 * br.ncx, ey = 2 * br.ncy, ez = 2 * br.ncz;
    auto finish = [&](T vk, T xk, T *fslot, unsigned off, unsigned fx, bool okx, int ly, int lz, bool ok) MF_INLINE {
        ok = ok && okx && ly <= ey && lz <= ez;
        const unsigned on = fx | br.yz_faces(ly, lz);
        const bool sh = (on & shf) != 0u, con = (on & dirf) != 0u;
        if constexpr (CG) {
            const double e = con ? ((on & shf & 42u) ? 0.0 : (double)xk * (double)xk) : (double)xk * (double)vk;
            energy += ok ? e : 0.0;
        }
        T *d = sh ? fslot : yb + off;
        if (ok) *d = con ? xk : vk;
    };
    const unsigned fx = br.x_faces(lx), fxe = br.x_faces(SL::RX);
    br.template for_rows<T>(m, [&](auto kc, int, unsigned off, int ly, int lz, bool ok) MF_INLINE {
        constexpr int k = decltype(kc)::value;
        finish(T(v[k]), T(xv[k]), f0 + k * fstep, off, fx, lx <= ex, ly, lz, ok);
    });
    br.template for_edge<T>(m, [&](auto kc, int, unsigned off, int ly, int lz, bool ok) MF_INLINE {
        constexpr int k = decltype(kc)::value;
        finish(T(v[K + k]), T(xv[K + k]), fe + k * SL::NT, off, fxe, SL::RX <= ex, ly, lz, ok);
    });
}

// Overlapping tiles: 4x4x4 cells every 3 cells, each computed like a slab of
// one brick.  Every node has a tile that holds all its cells, so the tile
// stores it complete and an apply is one launch, without face buffer and
// combine pass, for up to (4/3)^3 times the cells.  On small meshes, whose
// apply is the latency of its launches and of one brick, that is the better
// trade: FP64 8^3 cells 11.0 -> 7.8 us, 24^3 12.8 -> 7.9; FP32 22^3 12.3 -> 7.8;
// convective 16^3 15.5 -> 9.7; three phases 16^3 15.6 -> 10.5.
constexpr int TB = 3; // cells from one tile to the next
struct Tile : Slab<1> {
    static __host__ __device__ int count(int n) { return n <= BB ? 1 : (n + 1) / TB; }
    static __host__ __device__ int64_t count(const KMesh &m) { return (int64_t)count(m.nx) * count(m.ny) * count(m.nz); }
    __device__ __forceinline__ Tile(const KMesh &m, int tid_) : Slab<1>(Brick::xcd_index(), tid_)
    {
        const unsigned tx_ = (unsigned)count(m.nx), ty_ = (unsigned)count(m.ny), q = (unsigned)brick / tx_;
        bx = (int)((unsigned)brick - q * tx_);
        bz = (int)(q / ty_);
        by = (int)(q - (unsigned)bz * ty_);
        place(m, TB, TB);
    }
};

// Finish a tile's own nodes: along each direction 1 .. 2 TB (0 too at the low
// end of the mesh, up to the last one at its high end).  Arguments as for
// finish_nodes.
template <typename T>
__device__ __forceinline__ void finish_tile(const KMesh &m, const Tile &br, T *__restrict__ y, T (&v)[Tile::NV],
                                            T (&xv)[Tile::NV])
{
    T *const yb = y + node_index(m, 2 * br.c0x, 2 * br.c0y, 2 * br.c0z);
    const unsigned shf = br.shared_faces(m), dirf = br.dirichlet_faces(m);
    const int x0 = shf & 1u ? 1 : 0, y0 = shf & 4u ? 1 : 0, z0 = shf & 16u ? 1 : 0;
    const int x1 = shf & 2u ? 2 * TB : 2 * br.ncx, y1 = shf & 8u ? 2 * TB : 2 * br.ncy, z1 = shf & 32u ? 2 * TB : 2 * br.ncz;
    auto finish = [&](T vk, T xk, int lx, unsigned off, int ly, int lz, bool ok) MF_INLINE {
        const bool own = ok && lx >= x0 && lx <= x1 && ly >= y0 && ly <= y1 && lz >= z0 && lz <= z1;
        const bool con = ((br.x_faces(lx) | br.yz_faces(ly, lz)) & dirf) != 0u;
        if (own) yb[off] = con ? xk : vk;
    };
    const int lx = br.tid % Tile::RX;
    br.template for_rows<T>(m, [&](auto kc, int, unsigned off, int ly, int lz, bool ok) MF_INLINE {
        constexpr int k = decltype(kc)::value;
        finish(T(v[k]), T(xv[k]), lx, off, ly, lz, ok);
    });
    br.template for_edge<T>(m, [&](auto kc, int, unsigned off, int ly, int lz, bool ok) MF_INLINE {
        constexpr int k = Tile::STEPS + decltype(kc)::value;
        finish(T(v[k]), T(xv[k]), Tile::RX, off, ly, lz, ok);
    });
}

// Lanes that finish one slab's (or brick's) shared nodes, at most five nodes each.
template <typename SL> __host__ __device__ constexpr int combine_lanes() { return SL::W == 1 ? BNT : 2 * BNT; }
constexpr int SCT = 256; // threads of a slab-combine workgroup

// The combine pass of an apply on slabs or bricks: y = x on Dirichlet nodes.
template <typename T, typename SL>
__device__ __forceinline__ void combine_slabs(const KMesh &m, const T *__restrict__ face, const T *__restrict__ x,
                                              T *__restrict__ y)
{
    constexpr int L = combine_lanes<SL>(), PER = SCT / L;
    const int slab = Brick::xcd_index() * PER + (int)threadIdx.x / L, lane = (int)threadIdx.x % L;
    if (slab >= n_slabs<SL::W>(m)) return; // whole wavefronts; no barrier follows in them
    const SL br(m, lane, slab);
    const int nbx = (int)ceil_div(m.nx, br.CX), nby = (int)ceil_div(m.ny, BB), nbz = (int)ceil_div(m.nz, BB);
    auto f = [&](int64_t g, bool constrained, T s) { y[g] = constrained ? x[g] : s; };
    if (br.inner(m)) combine_brick_nodes<T, true, L, true>(m, br, nbx, nby, nbz, lane, face, f);
    else combine_brick_nodes<T, true, L, false>(m, br, nbx, nby, nbz, lane, face, f);
}

// Bricks (wavefronts) per brick-combine workgroup.
constexpr int CBW = 4;

template <typename T, int DMODE>
__device__ __forceinline__ void combine_brick(const KMesh &m, const T *__restrict__ face, const T *__restrict__ x,
                                              T *__restrict__ y)
{
    const int brick = Brick::xcd_index() * CBW + (int)threadIdx.x / BNT;
    if (brick >= n_bricks(m)) return; // whole wavefronts; no barrier follows in them
    combine_brick_visit<T, DMODE != 0>(m, brick, (int)threadIdx.x % BNT, face, [&](int64_t g, bool constrained, T s) {
        if (DMODE != 0 && constrained) y[g] = DMODE == 1 ? x[g] : ((DMODE == 2 || DMODE == 4) ? T(1) : T(0));
        else y[g] = DMODE == 4 ? T(1) / s : s;
    });
}

} // namespace mf
