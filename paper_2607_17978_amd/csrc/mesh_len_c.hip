// Mesh passes of the axis lengths of group c (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(80) X(96) X(216) X(480)
QEQ_LEN_GROUP(mesh_len_c, LENGTHS)
