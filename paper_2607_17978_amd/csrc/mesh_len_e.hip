// Mesh passes of the axis lengths of group e (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(16) X(36) X(160) X(256) X(400)
QEQ_LEN_GROUP(mesh_len_e, LENGTHS)
